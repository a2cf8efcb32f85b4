"""Forward calls that are one launch: operands and results must be the bytes of the quantiser and GEMM calls, which
other files pin to the oracle."""
import pytest
import torch

import paper_2605_09825_amd as mx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# one block; one element beyond a tile of rows and columns, columns in no whole 4; rows of 4, 5, 8, 9 and 16 blocks (each count of blocks per
# lane and its neighbour); 256 tiles (the most) and 257 (two launches); one block more per row than fits
@pytest.mark.parametrize("shape", [(1, 1, 32), (33, 35, 32), (32, 32, 128), (31, 66, 160), (65, 40, 256), (40, 67, 288), (7, 97, 480),
                                   (256, 512, 512), (512, 512, 64), (32, 32 * 257, 64), (96, 64, 544)])
@pytest.mark.parametrize("had,rnd", [(mx.HAD_NONE, mx.RNE), (mx.HAD_DET, mx.SR), (mx.HAD_RANDSIGN, mx.RNE), (mx.HAD_DET16, mx.RNE),
                                     (mx.HAD_RANDSIGN16, mx.SR)])
@pytest.mark.parametrize("out_dtype", [mx.OUT_BF16, mx.OUT_FP32])
def test_small_forward_equals_quantiser_and_gemm_calls(shape, had, rnd, out_dtype):
    M, N, K = shape
    print(f"[fwd small] M={M} N={N} K={K} had={had} rnd={rnd} out={out_dtype}", flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N + K)
    x = torch.randn((M, K), generator=g, device=DEV).to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device=DEV) * 0.02).to(torch.bfloat16)
    x[0, 0], w[N - 1, K - 1] = float("inf"), float("nan")  # (marked blocks: NaN in row 0 of Y and in its last column)
    cfg = mx.make_cfg(had, rnd, 77, y_dtype=out_dtype)
    y, ws = mx.mxfp4_linear_fwd(x, w, cfg)
    off = mx.mxfp4_linear_workspace_layout(M, N, K, False)
    xq, xs = mx.mxfp4_quantize(x, mx.AXIS_LAST, had, rnd, 77)
    wq, wsc = mx.mxfp4_quantize(w, mx.AXIS_LAST, had, rnd, 77 ^ (1 << 48))
    for o, t in zip(off, (xq, xs, wq, wsc)):
        assert torch.equal(ws[o:o + t.numel()], t.flatten())
    want = mx.mxfp4_gemm(xq, xs, wq, wsc, out_dtype=out_dtype)
    assert torch.equal(y.isnan(), want.isnan()) and torch.equal(y.nan_to_num(0.0), want.nan_to_num(0.0))


def test_small_forward_over_its_own_input():
    x = torch.randn((256, 256), device=DEV).to(torch.bfloat16)
    w = (torch.randn((256, 256), device=DEV) * 0.02).to(torch.bfloat16)
    cfg = mx.make_cfg(mx.HAD_DET, mx.RNE, 0)
    want, _ = mx.mxfp4_linear_fwd(x, w, cfg)
    mx.mxfp4_linear_fwd(x, w, cfg, y=x)
    assert torch.equal(x, want)
