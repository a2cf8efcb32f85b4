"""Backward calls whose three tensors are quantised in one launch: the operands must be the bytes of the single quantiser
calls, which other files pin to the oracle."""
import pytest
import torch

import paper_2605_09825_amd as mx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# one block; a last tile of one row block and of a few columns in each tensor; W and X of 496 tiles of 256 x 128, of 511 (the most in one launch, which
# tests/test_launch_limits.py pins) and of 512 (two launches, rounded to nearest; with stochastic rounding one)
@pytest.mark.parametrize("shape", [(32, 32, 8), (160, 288, 136), (416, 96, 264), (2080, 4320, 1440), (4096, 4096, 2048), (4096, 3840, 2048),
                                   (256, 18432, 896), (256, 16128, 1024)])
@pytest.mark.parametrize("had,rnd", [(mx.HAD_NONE, mx.RNE), (mx.HAD_RANDSIGN, mx.SR), (mx.HAD_DET16, mx.RNE)])
def test_backward_operands_equal_the_single_quantiser_calls(shape, had, rnd):
    M, N, K = shape
    print(f"[bwd operands] M={M} N={N} K={K} had={had} rnd={rnd}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N + K)
    x, w, dy = ((torch.randn(s, generator=g, device=DEV) * f).to(torch.bfloat16)
                for s, f in (((M, K), 1.0), ((N, K), 0.02), ((M, N), 1e-3)))
    _, _, ws = mx.mxfp4_linear_bwd(dy, x, w, mx.make_cfg(had, rnd, 77))
    off = mx.mxfp4_linear_workspace_layout(M, N, K, True)
    want = (mx.mxfp4_quantize(dy, mx.AXIS_LAST, had, rnd, 77 ^ (2 << 48)) + mx.mxfp4_quantize(w, mx.AXIS_FIRST, had, rnd, 77 ^ (3 << 48)) +
            mx.mxfp4_quantize(dy, mx.AXIS_FIRST, had, rnd, 77 ^ (4 << 48)) + mx.mxfp4_quantize(x, mx.AXIS_FIRST, had, rnd, 77 ^ (5 << 48)))
    for o, t in zip(off, want):
        assert torch.equal(ws[o:o + t.numel()], t.flatten())
