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


# Dgrad and Wgrad in one launch: on each tile shape, ragged everywhere, of very different lengths, one of them in whole
# tiles, scale arrays of less than 16 bytes; few narrow tiles of the one beside the other (Wgrad in 128 of them, all of Dgrad
# beside it or part of it behind it; Dgrad in 128); one after the other; MXFP8 as well; fp32 and bf16 dX, dW accumulated or not
@pytest.mark.parametrize("shape", [(32, 32, 8), (32, 32, 32), (64, 96, 160), (2048, 32, 64), (96, 2080, 1440), (2048, 768, 3072),
                                   (1056, 2080, 4320), (4096, 1024, 4096), (8192, 1024, 4096), (1024, 4096, 4096),
                                   (8192, 1024, 1024)])
@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
@pytest.mark.parametrize("dx_dtype,accumulate", [(mx.OUT_BF16, True), (mx.OUT_FP32, False)])
def test_backward_products_equal_the_single_gemm_calls(shape, fmt, dx_dtype, accumulate):
    M, N, K = shape
    print(f"[bwd products] M={M} N={N} K={K} fmt={fmt} dx={dx_dtype} accumulate={accumulate}", flush=True)
    x, w, dy = tensor(M, K, 1.0, 1), tensor(N, K, 0.02, 2), tensor(M, N, 1e-3, 3)
    kind = mx.mxfp4_gemm_pair_route((M, K, N), (N, K, M), (fmt, fmt), (dx_dtype, mx.OUT_FP32), accumulate)[0]
    whole = {(4096, 1024, 4096): mx.PAIR_NARROW_BESIDE_WIDE, (8192, 1024, 4096): mx.PAIR_NARROW_BESIDE_WIDE,
             (1024, 4096, 4096): mx.PAIR_NARROW_BESIDE_WIDE, (8192, 1024, 1024): mx.PAIR_APART}
    assert kind == (mx.PAIR_EDGE if fmt else whole.get(shape, mx.PAIR_EDGE))
    cfg = mx.make_cfg(mx.HAD_DET, mx.RNE, 5, dx_dtype=dx_dtype, dw_accumulate=accumulate, dgrad_format=fmt,
                      wgrad_format=fmt)
    dw0 = torch.randn((N, K), device=DEV)
    dx, dw, ws = mx.mxfp4_linear_bwd(dy, x, w, cfg, dw=dw0.clone())
    off = mx.mxfp4_linear_workspace_layout(M, N, K, True, cfg)

    def operand(i, R, C):
        row = C if fmt == mx.FMT_E4M3 else C // 2
        return (ws[off[i]:off[i] + R * row].view(R, row), ws[off[i + 1]:off[i + 1] + R * (C // 32)].view(R, C // 32))
    (gq, gs), (wq, wsc), (tq, ts), (xq, xs) = operand(0, M, N), operand(2, K, N), operand(4, N, M), operand(6, K, M)
    fmts = dict(a_format=fmt, b_format=fmt)
    assert torch.equal(dx, mx.mxfp4_gemm(gq, gs, wq, wsc, out_dtype=dx_dtype, **fmts))
    want = dw0.clone()
    mx.mxfp4_gemm(tq, ts, xq, xs, out=want, out_dtype=mx.OUT_FP32, accumulate=accumulate, **fmts)
    assert torch.equal(dw, want)


# the weight gradient alone: dY and X in one launch, or (X beyond the last-level cache, dY not) in two
@pytest.mark.parametrize("shape", [(32, 8, 8), (288, 136, 1000), (4096, 64, 32896)])
@pytest.mark.parametrize("rnd", [mx.RNE, mx.SR])
def test_wgrad_operands_equal_the_single_quantiser_calls(shape, rnd):
    M, N, K = shape
    print(f"[wgrad operands] M={M} N={N} K={K} rnd={rnd}", flush=True)
    x, dy = tensor(M, K, 1.0, 1), tensor(M, N, 1e-3, 3)
    cfg = mx.make_cfg(mx.HAD_RANDSIGN16, rnd, 99)
    _, dw, ws = mx.mxfp4_linear_bwd(dy, x, None, cfg, need_dx=False)
    off = mx.mxfp4_linear_workspace_layout(M, N, K, True)[4:]
    gq, gs = mx.mxfp4_quantize(dy, mx.AXIS_FIRST, mx.HAD_RANDSIGN16, rnd, 99 ^ (4 << 48))
    xq, xs = mx.mxfp4_quantize(x, mx.AXIS_FIRST, mx.HAD_RANDSIGN16, rnd, 99 ^ (5 << 48))
    for o, t in zip(off, (gq, gs, xq, xs)):
        assert torch.equal(ws[o:o + t.numel()], t.flatten())
    assert torch.equal(dw, mx.mxfp4_gemm(gq, gs, xq, xs, out_dtype=mx.OUT_FP32))


# Few narrow tiles of one product beside many wide ones of the other: (problem on narrow tiles, workgroups per XCD with one,
# tiles of the wide product that these add).  Tile counts in whole 8s and not (workgroups without a narrow tile), nothing, a
# round or two rounds or all of the wide product behind them; every combination of output types; each product first.
MIX = [((5632, 1280, 1024), (1024, 1280, 5632), 1, 5, 0), ((5376, 1280, 1280), (1280, 1280, 5376), 1, 7, 0),
       ((2048, 2560, 1280), (1280, 2560, 2048), 1, 13, 0), ((7424, 2304, 1792), (1792, 2304, 7424), 1, 16, 128),
       ((2048, 4352, 1024), (1024, 4352, 2048), 1, 17, 136), ((2816, 5632, 1280), (1280, 5632, 2816), 1, 28, 224),
       ((4352, 7936, 1024), (1024, 7936, 4352), 1, 31, 496)]


@pytest.mark.parametrize("case", MIX)
@pytest.mark.parametrize("swap", [False, True])
def test_narrow_beside_wide_equals_the_single_gemm_calls(case, swap):
    g = torch.Generator(device=DEV)
    g.manual_seed(case[3])

    def codes(R, C):
        return (torch.randint(0, 256, (R, C // 2), generator=g, device=DEV, dtype=torch.uint8),
                torch.randint(100, 150, (R, C // 32), generator=g, device=DEV, dtype=torch.uint8))
    shapes = case[1::-1] if swap else case[:2]
    ops = [(codes(Ra, C), codes(Rb, C)) for Ra, Rb, C in shapes]
    for dt0, dt1, acc in [(mx.OUT_BF16, mx.OUT_FP32, False), (mx.OUT_BF16, mx.OUT_FP32, True), (mx.OUT_BF16, mx.OUT_BF16, False),
                          (mx.OUT_FP32, mx.OUT_FP32, False), (mx.OUT_FP32, mx.OUT_FP32, True), (mx.OUT_FP32, mx.OUT_BF16, False)]:
        print(f"[mix] {shapes} dt={dt0},{dt1} acc={acc}", flush=True)
        route = mx.mxfp4_gemm_pair_route(*shapes, out_dtypes=(dt0, dt1), accumulate1=acc)
        assert route == (mx.PAIR_NARROW_BESIDE_WIDE, 0 if swap else case[2]) + case[3:]
        base = torch.full((shapes[1][0], shapes[1][1]), 0.5, dtype=torch.float32 if dt1 else torch.bfloat16, device=DEV)
        want0 = mx.mxfp4_gemm(*ops[0][0], *ops[0][1], out_dtype=dt0)
        want1 = mx.mxfp4_gemm(*ops[1][0], *ops[1][1], out=base.clone(), out_dtype=dt1, accumulate=acc)
        out0, out1 = torch.full_like(want0, 3.0), base.clone()
        mx.mxfp4_gemm_pair(*ops[0], out0, *ops[1], out1, accumulate1=acc)
        assert torch.equal(out0, want0) and torch.equal(out1, want1)


# the weight gradient of a few tokens, added to: 128 x 64 tiles at any size up to 512 tokens, in MXFP8 up to 256
@pytest.mark.parametrize("shape", [(32, 8384, 2784), (256, 4128, 2080), (512, 8192, 2304), (544, 8192, 2304)])
@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
def test_weight_gradients_of_a_few_tokens_added_to(shape, fmt):
    M, N, K = shape
    _, _, tile, _ = mx.mxfp4_gemm_pair_route((M, K, N), (N, K, M), (fmt, fmt), (mx.OUT_BF16, mx.OUT_FP32), True)
    assert (tile == 1) == (M <= (256 if fmt else 512))
    test_backward_products_equal_the_single_gemm_calls(shape, fmt, mx.OUT_BF16, True)
