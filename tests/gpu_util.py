"""Helpers shared by the GPU parity tests: move seeded host tensors to the device, call the
library through its Python binding (= the C ABI), bring results back as numpy."""
import numpy as np
import torch

import paper_2605_09825_amd as mx
from paper_2605_09825_amd import synth


def dev():
    return torch.device("cuda:0")


def to_gpu_bf16(t_cpu: torch.Tensor) -> torch.Tensor:
    assert t_cpu.dtype == torch.bfloat16
    return t_cpu.to(dev())


def gpu_quantize(t_cpu: torch.Tensor, axis=mx.AXIS_LAST, had=mx.HAD_NONE, rnd=mx.RNE, seed=0):
    """Quantise a CPU bf16 tensor (possibly a strided row view) on the GPU; numpy (q, s) back."""
    if t_cpu.is_contiguous():
        x = to_gpu_bf16(t_cpu)
    else:  # keep the leading dimension: copy the base storage, then take the same view
        base = t_cpu._base
        assert base is not None and base.dim() == 2
        off = t_cpu.storage_offset() - base.storage_offset()
        r0, c0 = divmod(off, base.stride(0))
        x = to_gpu_bf16(base)[r0:r0 + t_cpu.shape[0], c0:c0 + t_cpu.shape[1]]
    q, s = mx.mxfp4_quantize(x, axis, had, rnd, seed)
    torch.cuda.synchronize()
    return q.cpu().numpy(), s.cpu().numpy()


def first_mismatch(a: np.ndarray, b: np.ndarray) -> str:
    if a.shape != b.shape:
        return f"shape {a.shape} vs {b.shape}"
    bad = np.argwhere(a != b)
    if bad.size == 0:
        return "equal"
    i = tuple(bad[0])
    return f"{len(bad)} of {a.size} differ; first at {i}: gpu {a[i]:#x} vs oracle {b[i]:#x}"


def assert_runs_on(kernel, Ra, Rb, C, fmt=0, **kw):
    """The kernel that a product of this shape runs on is the one that the test is about (kernel: a name below)."""
    routes = {"any": mx.ROUTE_ANY_SHAPE, "64x64": mx.ROUTE_EDGE_64, "128x64": mx.ROUTE_EDGE_128,
              "128x256": mx.ROUTE_EDGE_256, "moved back": mx.ROUTE_RAGGED_TILED}
    kinds = {"wide": mx.GEMM_TILED_256, "narrow": mx.GEMM_TILED_128, "tail": mx.GEMM_TILED_256_TAIL_128}
    got = mx.mxfp4_gemm_route(Ra, Rb, C, fmt, fmt, **kw)
    assert got == routes.get(kernel, mx.ROUTE_BLOCKS), (kernel, got)
    if kernel in kinds:
        plan = mx.mxfp4_gemm_plan(Ra, Rb, C, fmt, fmt)
        assert len(plan) == 1 and plan[0][0] == kinds[kernel], (kernel, plan)
