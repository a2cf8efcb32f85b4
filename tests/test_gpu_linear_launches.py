"""GPU parity of the linear calls whose quantisations or products share a launch: the bytes and results must be those
of the single-operand calls, which other files pin to the oracle."""
import pytest
import torch

import paper_2605_09825_amd as mx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def tensor(rows, cols, std, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return (torch.randn((rows, cols), generator=g, device=DEV) * std).to(torch.bfloat16)


# one block, a last workgroup with one block, X or W much the smaller, W beyond the last-level cache and X not (each
# tensor then keeps a launch, and a store policy, of its own)
@pytest.mark.parametrize("shape", [(1, 8, 32), (257, 8, 32), (8, 1000, 96), (3, 32800, 4096)])
@pytest.mark.parametrize("rnd", [mx.RNE, mx.SR])
def test_forward_operands_equal_the_single_quantiser_calls(shape, rnd):
    M, N, K = shape
    print(f"[fwd operands] M={M} N={N} K={K} rnd={rnd}", flush=True)
    x, w = tensor(M, K, 1.0, 1), tensor(N, K, 0.02, 2)
    cfg = mx.make_cfg(mx.HAD_RANDSIGN, rnd, 77)
    y, ws = mx.mxfp4_linear_fwd(x, w, cfg)
    off = mx.mxfp4_linear_workspace_layout(M, N, K, False)
    xq, xs = mx.mxfp4_quantize(x, mx.AXIS_LAST, mx.HAD_RANDSIGN, rnd, 77)
    wq, wsc = mx.mxfp4_quantize(w, mx.AXIS_LAST, mx.HAD_RANDSIGN, rnd, 77 ^ (1 << 48))
    for o, t in zip(off, (xq, xs, wq, wsc)):
        assert torch.equal(ws[o:o + t.numel()], t.flatten())
    assert torch.equal(y, mx.mxfp4_gemm(xq, xs, wq, wsc, out_dtype=mx.OUT_BF16))
