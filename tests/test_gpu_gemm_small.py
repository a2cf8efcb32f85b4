"""GPU tests: the ragged-shape kernel's 32 x 32 tiles (outputs of up to 512 of them): edges of tiles, rows of the scale arrays at every
alignment, last stages of one block up to whole, arrays of less than 8 scale bytes, both numbers of stage buffers, two products in a launch; with
them sizes that are faster on 64 x 64 tiles (rows of less than a stage)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_09825_amd as mx
import test_gpu_linear_launches as launches
from gpu_util import edge_kernel
from test_gpu_fp8 import rand_fp4, rand_fp8
from test_gpu_gemm import gpu

pytestmark = pytest.mark.gpu

# rows, columns, C: E2M1 stages hold 8 blocks of 32, E4M3 stages 4; batches of scale bytes 64
SHAPES = [(33, 64, 64), (1, 33, 544), (33, 36, 288), (64, 33, 256), (32, 32, 2080), (65, 97, 2016), (3, 70, 4128),
          (24, 500, 4320), (3, 68, 64), (100, 36, 8160), (511, 1000, 608), (257, 256, 1024)]


def operands(rows, C, fmt, seed):
    rng = np.random.default_rng(seed)
    q = rng.integers(0, 256, (rows, C // 2 if fmt == mx.FMT_E2M1 else C), dtype=np.uint8)
    if fmt == mx.FMT_E4M3:
        q = (q & 0x80) | (q & 0x07) | 0x38  # magnitudes 1 .. 1.875: no bits of a product are dropped
    return q, rng.integers(120, 131, (rows, C // 32), dtype=np.uint8)


@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
@pytest.mark.parametrize("shape", SHAPES)
def test_against_the_oracle(shape, fmt):
    Ra, Rb, C = shape
    fmts = dict(a_format=fmt, b_format=fmt)
    ld = Rb + 1 + Ra % 4
    if (Ra + 31) // 32 * ((Rb + 31) // 32) > 1:  # (of the short ones at least one call: the others are the any-shape kernel's)
        assert mx.ROUTE_EDGE_64 in [mx.mxfp4_gemm_route(Ra, Rb, C, out_dtype=mx.OUT_FP32, **fmts), mx.mxfp4_gemm_route(
            Ra, Rb, C, ld_out=ld, out_dtype=mx.OUT_FP32, accumulate=True, **fmts)]
    (aq, as_), (bq, bs) = operands(Ra, C, fmt, 1), operands(Rb, C, fmt, 2)
    want, absum = oracle.gemm_fmt(aq, as_, fmt, bq, bs, fmt)
    canvas = torch.full((Ra, ld), 0.5, device="cuda:0")
    a, sa, b, sb = gpu(aq), gpu(as_), gpu(bq), gpu(bs)
    mx.mxfp4_gemm(a, sa, b, sb, out=canvas[:, :Rb], accumulate=True, **fmts)
    dense = mx.mxfp4_gemm(a, sa, b, sb, **fmts)
    half = mx.mxfp4_gemm(a, sa, b, sb, out_dtype=mx.OUT_BF16, **fmts)
    assert (np.abs(dense.cpu().numpy().astype(np.float64) - want) <= 1e-5 * absum).all()  # the bound of the public contract
    assert torch.equal(canvas[:, :Rb], dense + 0.5) and bool((canvas[:, Rb:] == 0.5).all())
    assert torch.equal(half, dense.to(torch.bfloat16))


@pytest.mark.parametrize("shapes", [((33, 70, 480), (65, 36, 4128)), ((200, 96, 2016), (96, 128, 224))])
def test_two_products_in_a_launch(shapes):
    assert mx.mxfp4_gemm_pair_route(*shapes)[:1] + mx.mxfp4_gemm_pair_route(*shapes)[2:3] == (mx.PAIR_EDGE, 0)
    ops, outs = [], []
    for n, (Ra, Rb, C) in enumerate(shapes):
        ops.append([tuple(map(gpu, operands(R, C, mx.FMT_E2M1, 10 * n + R))) for R in (Ra, Rb)])
        outs.append(torch.empty((Ra, Rb), device="cuda:0", dtype=(torch.bfloat16, torch.float32)[n]))
    mx.mxfp4_gemm_pair(*ops[0], outs[0], *ops[1], outs[1])
    for ((a, sa), (b, sb)), out in zip(ops, outs):
        single = mx.mxfp4_gemm(a, sa, b, sb, out_dtype=mx.OUT_FP32 if out.dtype == torch.float32 else mx.OUT_BF16)
        assert torch.equal(out, single)


@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
@pytest.mark.parametrize("C", [4128, 8160, 14336])
@pytest.mark.parametrize("rows", [100, 500])  # one workgroup per compute unit and eight stage buffers; two and four
def test_more_batches_of_scale_bytes_than_buffers(rows, C, fmt):
    # scale bytes over 2^50: one taken from another batch shows.  The same rows among more of them run on 64 x 64 tiles, bit for bit
    rng = np.random.default_rng(C + rows + fmt)
    def operand(R):
        q = rng.integers(0, 256, (R, C // 2 if fmt == mx.FMT_E2M1 else C), dtype=np.uint8)
        return gpu(q & 0xF7 if fmt == mx.FMT_E4M3 else q), gpu(rng.integers(100, 150, (R, C // 32), dtype=np.uint8))
    (aq, as_), (bq, bs) = operand(1000), operand(1000)
    kw = dict(a_format=fmt, b_format=fmt, out_dtype=mx.OUT_FP32)
    assert mx.mxfp4_gemm_route(1000, 1000, C, fmt, fmt, ld_out=1001) == mx.ROUTE_EDGE_64
    out = [torch.empty((R, 1001), device="cuda:0") for R in (rows, 1000)]
    for o in out:
        mx.mxfp4_gemm(aq[:len(o)], as_[:len(o)], bq, bs, out=o[:, :1000], **kw)
    assert torch.equal(out[0][:, :1000], out[1][:rows, :1000])


# the fewest stages that run on these tiles: whole, and with a ragged last one, up to 256 tiles and beyond; arrays of less than 8 scale bytes
@pytest.mark.parametrize("shape,fmt", [((64, 33, 256), mx.FMT_E2M1), ((33, 36, 288), mx.FMT_E2M1), ((500, 512, 480), mx.FMT_E2M1),
                                       ((511, 1000, 512), mx.FMT_E2M1), ((511, 1000, 1056), mx.FMT_E2M1), ((33, 64, 128), mx.FMT_E4M3),
                                       ((33, 36, 288), mx.FMT_E4M3), ((500, 510, 352), mx.FMT_E4M3), ((511, 1000, 256), mx.FMT_E4M3),
                                       ((511, 1000, 928), mx.FMT_E4M3), ((1, 100, 128), mx.FMT_E4M3)])
def test_fewest_stages(shape, fmt):
    Ra, Rb, _ = shape
    call = dict(shape=shape, fmt=fmt, out_dtype=mx.OUT_FP32)
    assert "32x32" in (edge_kernel(call), edge_kernel(dict(call, ld=Rb + 1 + Ra % 4, accumulate=True)))
    test_against_the_oracle(shape, fmt)


# Each product alone runs on 32 x 32 tiles, the pair, of more than 512 of them, on 64 x 64 ones: another matrix instruction, the same bits
@pytest.mark.parametrize("shapes", [((640, 640, 1024), (640, 640, 2048)), ((608, 608, 1440), (608, 608, 1440)), ((512, 1000, 4128), (1000, 300, 512))])
def test_pairs_beside_single_products(shapes):
    products = [dict(shape=s, out_dtype=d) for s, d in zip(shapes, (mx.OUT_BF16, mx.OUT_FP32))]
    assert [edge_kernel(p) for p in products] == ["32x32", "32x32"] and edge_kernel(*products) == "64x64"
    rng = np.random.default_rng(sum(shapes[0]))
    ops = [[tuple(map(gpu, rand_fp4(rng, R, C))) for R in (Ra, Rb)] for Ra, Rb, C in shapes]
    outs = [torch.empty(s[:2], device="cuda:0", dtype=t) for s, t in zip(shapes, (torch.bfloat16, torch.float32))]
    mx.mxfp4_gemm_pair(*ops[0], outs[0], *ops[1], outs[1])
    for ((a, sa), (b, sb)), out, p in zip(ops, outs, products):
        assert torch.equal(out, mx.mxfp4_gemm(a, sa, b, sb, out_dtype=p["out_dtype"]))


def test_backward_pairs_beside_single_products():
    M = N = K = 640
    product = dict(shape=(M, N, K), fmt=mx.FMT_E4M3)
    assert edge_kernel(product) == "32x32" and edge_kernel(product, dict(product, out_dtype=mx.OUT_FP32)) == "64x64"
    launches.test_backward_products_equal_the_single_gemm_calls((M, N, K), mx.FMT_E4M3, mx.OUT_BF16, False)


@pytest.mark.parametrize("C", [512, 1440, 4096])
@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
def test_any_codes_as_on_larger_tiles(C, fmt):
    rng = np.random.default_rng(C + fmt)
    (aq, sa), (bq, sb) = [tuple(map(gpu, (rand_fp8 if fmt else rand_fp4)(rng, R, C))) for R in (1500, 640)]
    kw = dict(a_format=fmt, b_format=fmt, out_dtype=mx.OUT_FP32)
    assert [edge_kernel(dict(shape=(R, 640, C), fmt=fmt, out_dtype=mx.OUT_FP32, ld=641)) for R in (640, 1500)] == ["32x32", "64x64"]
    out = [torch.empty((R, 641), device="cuda:0") for R in (640, 1500)]
    for o in out:
        mx.mxfp4_gemm(aq[:len(o)], sa[:len(o)], bq, sb, out=o[:, :640], **kw)
    assert torch.equal(out[0][:, :640], out[1][:640, :640])
