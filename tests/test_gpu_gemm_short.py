"""GPU tests: products of at most 256 bytes of codes per row with more than 512 tiles of 64 x 64, on the short-row kernel where rows of the output are
in no whole cache lines, beside the general one on the same tiles: ragged edges of the 128 x 64 tiles, one and two stages in whole and in part, every
way of storing (rows of whole cache lines, 16, 8, 4 bytes and single elements), more than 4096 tiles, two products in a launch."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_09825_amd as mx
from gpu_util import assert_runs_on, edge_kernel
from test_gpu_fp8 import FP8_RTOL, rand_fp4, rand_fp8
from test_gpu_gemm import RTOL, gpu

pytestmark = pytest.mark.gpu

SHAPES = [(1300, 1700, 32), (2113, 1023, 96), (1281, 1729, 256), (1300, 1728, 288), (1407, 1601, 480), (1280, 1792, 512)]


@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_output_once_and_nothing_outside(shape, fmt):
    Ra, Rb, C = shape
    C = C if fmt == mx.FMT_E2M1 else (C // 2 + 31) // 32 * 32
    rng = np.random.default_rng(Ra + Rb + C + fmt)
    (aq, as_), (bq, bs) = [(rand_fp8 if fmt else rand_fp4)(rng, R, C) for R in (Ra, Rb)]
    want, absum = oracle.gemm_fmt(aq, as_, fmt, bq, bs, fmt)
    args = [gpu(t) for t in (aq, as_, bq, bs)]
    fmts = dict(a_format=fmt, b_format=fmt)
    first = None
    for ld in ((Rb + 63) // 64 * 64, (Rb + 7) // 8 * 8 + 8, (Rb + 3) // 8 * 8 + 4, Rb // 2 * 2 + 2, Rb // 2 * 2 + 1):
        ld += 8 if ld < Rb else 0
        assert_runs_on("128x64", Ra, Rb, C, fmt, ld_out=ld)
        canvas = torch.full((Ra + 1, ld), 7.0, dtype=torch.float32, device="cuda:0")
        mx.mxfp4_gemm(*args, out=canvas[:Ra, :Rb], out_dtype=mx.OUT_FP32, **fmts)
        got = canvas[:Ra, :Rb].clone()
        if first is None:
            first = got
            assert np.all(np.abs(got.cpu().numpy() - want) <= (FP8_RTOL if fmt else RTOL) * absum)
        assert torch.equal(got, first)
        mx.mxfp4_gemm(*args, out=canvas[:Ra, :Rb], out_dtype=mx.OUT_FP32, accumulate=True, **fmts)
        assert torch.equal(canvas[:Ra, :Rb], first + first)
        half = torch.full((Ra + 1, ld), 7.0, dtype=torch.bfloat16, device="cuda:0")
        mx.mxfp4_gemm(*args, out=half[:Ra, :Rb], out_dtype=mx.OUT_BF16, **fmts)
        assert torch.equal(half[:Ra, :Rb], first.to(torch.bfloat16))
        for c in (canvas, half):
            assert bool((c[:Ra, Rb:] == 7.0).all()) and bool((c[Ra] == 7.0).all())


def test_two_products_in_a_launch():
    shapes = ((1000, 1700, 288), (1300, 700, 64))
    assert mx.mxfp4_gemm_pair_route(*shapes)[0] == mx.PAIR_EDGE and mx.mxfp4_gemm_pair_route(*shapes)[2] == 1
    rng = np.random.default_rng(7)
    ops = [[tuple(gpu(t) for t in rand_fp4(rng, R, C)) for R in (Ra, Rb)] for Ra, Rb, C in shapes]
    outs = [torch.empty(s[:2], device="cuda:0", dtype=dt) for s, dt in zip(shapes, (torch.bfloat16, torch.float32))]
    mx.mxfp4_gemm_pair(*ops[0], outs[0], *ops[1], outs[1])
    for ((a, sa), (b, sb)), out in zip(ops, outs):
        assert torch.equal(out, mx.mxfp4_gemm(a, sa, b, sb, out_dtype=mx.OUT_FP32 if out.dtype == torch.float32 else mx.OUT_BF16))


# The short-row kernel alone, named by the rule that the launch asks: rows of whole cache lines take more than 4096 tiles.  Bit for bit the product of
# the same rows in two halves of fewer tiles, of which the oracle has a sample; and nothing outside
@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
@pytest.mark.parametrize("stages", [1, 2])
def test_whole_cache_lines(stages, fmt):
    Ra, Rb, C = 8200, 4160, ((224, 480), (96, 224))[fmt][stages - 1]
    rng = np.random.default_rng(C + fmt)
    (aq, as_), (bq, bs) = [(rand_fp8 if fmt else rand_fp4)(rng, R, C) for R in (Ra, Rb)]
    a, sa, b, sb = [gpu(t) for t in (aq, as_, bq, bs)]
    fmts = dict(a_format=fmt, b_format=fmt)
    rows = np.sort(rng.choice(Ra, 24, replace=False))
    rows[-1] = Ra - 1
    want, absum = oracle.gemm_fmt(aq[rows], as_[rows], fmt, bq, bs, fmt)
    ref = torch.empty((Ra, Rb), device="cuda:0")
    for r0, r1 in ((0, 4096), (4096, Ra)):
        assert edge_kernel(dict(shape=(r1 - r0, Rb, C), fmt=fmt, out_dtype=mx.OUT_FP32)) != "short"
        mx.mxfp4_gemm(a[r0:r1], sa[r0:r1], b, sb, out=ref[r0:r1], **fmts)
    assert np.all(np.abs(ref[torch.from_numpy(rows)].cpu().numpy() - want) <= (FP8_RTOL if fmt else RTOL) * absum)
    for dtype, code in ((torch.float32, mx.OUT_FP32), (torch.bfloat16, mx.OUT_BF16)):
        canvas = torch.full((Ra + 1, Rb), 7.0, dtype=dtype, device="cuda:0")
        call = dict(shape=(Ra, Rb, C), fmt=fmt, out_dtype=code)
        assert edge_kernel(call) == "short"
        mx.mxfp4_gemm(a, sa, b, sb, out=canvas[:Ra], out_dtype=code, **fmts)
        assert torch.equal(canvas[:Ra], ref.to(dtype)) and bool((canvas[Ra] == 7.0).all())
        if code == mx.OUT_FP32:
            assert edge_kernel(dict(call, accumulate=True)) == "short"
            mx.mxfp4_gemm(a, sa, b, sb, out=canvas[:Ra], out_dtype=code, accumulate=True, **fmts)
            assert torch.equal(canvas[:Ra], ref + ref) and bool((canvas[Ra] == 7.0).all())


# added to on the short-row kernel (more than 512 tiles), rows of 16 bytes and of single elements, beside the general kernels just off its range
@pytest.mark.parametrize("Ra,C,ld,kernel", [(8300, 96, 516, "short"), (8300, 480, 516, "short"), (8300, 96, 515, "short"), (8300, 96, 512, "128x64"),
                                            (8100, 96, 516, "128x64"), (8100, 480, 515, "128x64"), (12300, 480, 516, None), (16300, 480, 515, None)])
def test_added_to(Ra, C, ld, kernel):
    Rb = 510
    rng = np.random.default_rng(Ra + C + ld)
    (a, sa), (b, sb) = [tuple(gpu(t) for t in rand_fp4(rng, R, C)) for R in (Ra, Rb)]
    ran = edge_kernel(dict(shape=(Ra, Rb, C), out_dtype=mx.OUT_FP32, ld=ld, accumulate=True))
    assert ran == kernel if kernel else ran != "short"
    start = torch.randn((Ra + 1, ld), device="cuda:0")
    canvas = start.clone()
    mx.mxfp4_gemm(a, sa, b, sb, out=canvas[:Ra, :Rb], accumulate=True)
    product = torch.empty((Ra, 516), dtype=torch.float32, device="cuda:0")  # (not added to: the short-row kernel at any of these sizes but one)
    mx.mxfp4_gemm(a, sa, b, sb, out=product[:, :Rb])
    assert torch.equal(canvas[:Ra, :Rb], start[:Ra, :Rb] + product[:, :Rb])
    assert torch.equal(canvas[:Ra, Rb:], start[:Ra, Rb:]) and torch.equal(canvas[Ra], start[Ra])
