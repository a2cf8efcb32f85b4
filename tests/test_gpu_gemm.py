"""GPU parity of mxfp4_gemm against the CPU oracle (plain fp64 sum of decoded products).
Tolerance, written out: |gpu - oracle| <= 1e-5 * sum_c |a_c||b_c| on the fp32 output."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_09825_amd as mx
from paper_2605_09825_amd import synth
from gpu_util import assert_runs_on

pytestmark = pytest.mark.gpu
RTOL = 1e-5


def rand_operand(rng, R, C, s_lo=115, s_hi=135):
    q = rng.integers(0, 256, size=(R, C // 2), dtype=np.uint8)
    s = rng.integers(s_lo, s_hi, size=(R, C // 32), dtype=np.uint8)
    return q, s


def gpu(t):
    return torch.from_numpy(np.ascontiguousarray(t)).to("cuda:0")


def run_gemm(aq, as_, bq, bs, **kw):
    out = mx.mxfp4_gemm(gpu(aq), gpu(as_), gpu(bq), gpu(bs), **kw)
    torch.cuda.synchronize()
    return out


def assert_close(got, want, absum):
    err = np.abs(got.astype(np.float64) - want)
    bound = RTOL * absum
    worst = np.argmax(err - bound)
    assert (err <= bound).all(), (f"max err/absum {np.max(err / np.maximum(absum, 1e-300)):.3e}; "
                                  f"at {np.unravel_index(worst, err.shape)} got {got.flat[worst]} want {want.flat[worst]}")


@pytest.mark.parametrize("shape", [(64, 64, 128), (16, 16, 32), (37, 53, 96), (1, 1, 32), (256, 512, 512),
                                   (130, 70, 1024), (512, 384, 4096), (100, 260, 160), (512, 768, 1536),
                                   (256, 256, 1024), (768, 512, 2560), (512, 256, 1280), (256, 768, 1792)])
def test_random_codes_fp32(shape):
    Ra, Rb, C = shape
    rng = np.random.default_rng(Ra * 7 + Rb * 3 + C)
    aq, as_ = rand_operand(rng, Ra, C)
    bq, bs = rand_operand(rng, Rb, C)
    want, absum = oracle.gemm(aq, as_, bq, bs)
    got = run_gemm(aq, as_, bq, bs, out_dtype=mx.OUT_FP32).cpu().numpy()
    assert_close(got, want, absum)


@pytest.mark.parametrize("shape", [(300, 520, 1024), (544, 784, 1536), (320, 256, 2048), (256, 257, 1024),
                                   (1030, 513, 1024), (300, 520, 1280)])
def test_ragged_rows_and_columns_around_whole_tiles(shape):
    # row / column counts that leave edge strips beside a 256-aligned interior (different kernels write the
    # interior and the strips): every output element once, nothing outside
    Ra, Rb, C = shape
    rng = np.random.default_rng(Ra * 5 + Rb * 11 + C)
    aq, as_ = rand_operand(rng, Ra, C)
    bq, bs = rand_operand(rng, Rb, C)
    want, absum = oracle.gemm(aq, as_, bq, bs)
    ld = Rb + 8 - Rb % 8 + 8  # padded rows: the padding must stay untouched
    canvas = torch.full((Ra + 1, ld), 7.0, dtype=torch.float32, device="cuda:0")
    mx.mxfp4_gemm(gpu(aq), gpu(as_), gpu(bq), gpu(bs), out=canvas[:Ra, :Rb], out_dtype=mx.OUT_FP32)
    torch.cuda.synchronize()
    c = canvas.cpu().numpy()
    assert_close(c[:Ra, :Rb], want, absum)
    assert np.all(c[:Ra, Rb:] == 7.0) and np.all(c[Ra] == 7.0)
    # accumulate on top, and bf16 output = RNE of the fp32 result
    mx.mxfp4_gemm(gpu(aq), gpu(as_), gpu(bq), gpu(bs), out=canvas[:Ra, :Rb], out_dtype=mx.OUT_FP32, accumulate=True)
    b16 = run_gemm(aq, as_, bq, bs, out_dtype=mx.OUT_BF16)
    torch.cuda.synchronize()
    first = torch.from_numpy(c[:Ra, :Rb].copy())
    assert torch.equal(canvas[:Ra, :Rb].cpu(), first + first)
    assert torch.equal(b16.cpu(), first.to(torch.bfloat16))


def as_f32(want):
    """The oracle's fp64 value as the fp32 the kernel must deliver when the sum itself is exact: round to nearest
    even, gradual underflow, overflow to infinity."""
    with np.errstate(over="ignore"):
        return want.astype(np.float32)


@pytest.mark.parametrize("shape,kernel", [((64, 48, 32), "64x64"), ((30, 48, 32), "any"), ((256, 256, 1024), "64x64"),
                                          ((4096, 4096, 1024), "wide"), ((2048, 2560, 1024), "narrow"),
                                          ((4352, 4352, 1024), "tail"), ((4200, 4104, 1056), "moved back")])
def test_wide_scale_range_and_exactness_on_small_sums(shape, kernel):
    # one live block per row: at most 32 products, partial sums < 2^24 in units of the smallest product, so the
    # fp32 result must be exact -- also where it is a subnormal number (the matrix unit does not flush them) or
    # overflows (to infinity).  Scale bytes 60..200 put results between 2^-136 and beyond 2^128.
    Ra, Rb, C = shape
    assert_runs_on(kernel, Ra, Rb, C, out_dtype=mx.OUT_FP32)
    rng = np.random.default_rng(1)
    aq, as_ = rand_operand(rng, Ra, C, 60, 200)
    bq, bs = rand_operand(rng, Rb, C, 60, 190)
    aq[:, 16:] = 0  # (longer rows: every block but the first holds zero codes)
    want, _ = oracle.gemm(aq, as_, bq, bs)
    w32 = as_f32(want)
    tiny = float(np.finfo(np.float32).tiny)
    assert ((np.abs(want) < tiny) & (want != 0)).sum() > 0 and np.isinf(w32).sum() > 0  # both regimes are present
    got = run_gemm(aq, as_, bq, bs, out_dtype=mx.OUT_FP32).cpu().numpy()
    bad = np.argwhere(got != w32)
    assert bad.size == 0, (len(bad), bad[0], got[tuple(bad[0])], want[tuple(bad[0])])


def test_results_in_the_subnormal_range_are_not_flushed():
    # scale bytes 54..65 on both sides: every result is a multiple of 2^-148 (so fp32 holds it exactly), three in
    # four of them below fp32's smallest normal number
    rng = np.random.default_rng(4)
    aq, as_ = rand_operand(rng, 96, 32, 54, 66)
    bq, bs = rand_operand(rng, 80, 32, 54, 66)
    want, _ = oracle.gemm(aq, as_, bq, bs)
    tiny = float(np.finfo(np.float32).tiny)
    assert ((np.abs(want) < tiny) & (want != 0)).mean() > 0.5
    got = run_gemm(aq, as_, bq, bs, out_dtype=mx.OUT_FP32).cpu().numpy()
    assert np.array_equal(got.astype(np.float64), want)


@pytest.mark.parametrize("shape,kernel", [((64, 48, 96), "64x64"), ((30, 48, 96), "any"), ((512, 256, 1024), "64x64"),
                                          ((4096, 4096, 1024), "wide"), ((2048, 2560, 1024), "narrow"),
                                          ((4352, 4352, 1024), "tail")])
@pytest.mark.parametrize("out_dtype", [mx.OUT_FP32, mx.OUT_BF16])
def test_scale_byte_ff_gives_nan(shape, kernel, out_dtype):
    # 0xFF is the NaN of the E8M0 scale format (the quantiser writes it for a block that held a NaN or an
    # infinity, with all codes 0): every output whose row of A or row of B contains such a block is NaN, whatever
    # the codes under it, and nothing else is
    Ra, Rb, C = shape
    assert_runs_on(kernel, Ra, Rb, C, out_dtype=out_dtype)
    rng = np.random.default_rng(8)
    aq, as_ = rand_operand(rng, Ra, C)
    bq, bs = rand_operand(rng, Rb, C)
    as_[3, 0] = 0xFF                       # live codes under the NaN scale
    as_[Ra - 2, C // 32 - 1] = 0xFF
    aq[Ra - 2, -16:] = 0                   # zero codes under it, as the quantiser leaves them
    bs[7, 1] = 0xFF
    want, absum = oracle.gemm(aq, as_, bq, bs)
    nan_want = np.isnan(want)
    assert nan_want[3].all() and nan_want[Ra - 2].all() and nan_want[:, 7].all()
    assert nan_want.sum() == 2 * Rb + Ra - 2
    got = run_gemm(aq, as_, bq, bs, out_dtype=out_dtype).float().cpu().numpy()
    assert np.array_equal(np.isnan(got), nan_want)
    ok = ~nan_want
    tol = 1e-5 * absum[ok] + (2.0 ** -8 * np.abs(want[ok]) if out_dtype == mx.OUT_BF16 else 0.0)
    assert (np.abs(got[ok] - want[ok]) <= tol).all()


def test_bf16_output_is_rne_of_the_fp32_output():
    rng = np.random.default_rng(2)
    aq, as_ = rand_operand(rng, 96, 256)
    bq, bs = rand_operand(rng, 80, 256)
    f32 = run_gemm(aq, as_, bq, bs, out_dtype=mx.OUT_FP32)
    b16 = run_gemm(aq, as_, bq, bs, out_dtype=mx.OUT_BF16)
    assert b16.dtype == torch.bfloat16
    want_bits = oracle.f32_to_bf16_rne(f32.cpu().numpy())
    got_bits = b16.cpu().view(torch.int16).numpy().view(np.uint16)
    assert np.array_equal(got_bits, want_bits)
    assert torch.equal(b16, f32.to(torch.bfloat16))


def test_accumulate_and_leading_dimension():
    rng = np.random.default_rng(3)
    aq, as_ = rand_operand(rng, 70, 128)
    bq, bs = rand_operand(rng, 50, 128)
    want, absum = oracle.gemm(aq, as_, bq, bs)
    big = torch.full((70, 64), 7.0, dtype=torch.float32, device="cuda:0")
    view = big[:, :50]
    mx.mxfp4_gemm(gpu(aq), gpu(as_), gpu(bq), gpu(bs), out=view, out_dtype=mx.OUT_FP32, accumulate=True)
    torch.cuda.synchronize()
    got = big.cpu().numpy()
    assert (got[:, 50:] == 7.0).all()                      # padding untouched
    assert_close(got[:, :50] - 7.0, want, absum + 1e-6 * 7.0 / RTOL)
    mx.mxfp4_gemm(gpu(aq), gpu(as_), gpu(bq), gpu(bs), out=view, out_dtype=mx.OUT_FP32, accumulate=False)
    torch.cuda.synchronize()
    assert_close(big.cpu().numpy()[:, :50], want, absum)


def test_empty_and_zero_length_contraction():
    e = torch.empty((0, 16), dtype=torch.uint8, device="cuda:0")
    es = torch.empty((0, 1), dtype=torch.uint8, device="cuda:0")
    b = torch.zeros((8, 16), dtype=torch.uint8, device="cuda:0")
    bs = torch.full((8, 1), 127, dtype=torch.uint8, device="cuda:0")
    assert mx.mxfp4_gemm(e, es, b, bs).shape == (0, 8)
    assert mx.mxfp4_gemm(b, bs, e, es).shape == (8, 0)
    # C = 0: the empty sum
    a0 = torch.empty((5, 0), dtype=torch.uint8, device="cuda:0")
    b0 = torch.empty((6, 0), dtype=torch.uint8, device="cuda:0")
    out = mx.mxfp4_gemm(a0, a0, b0, b0)
    torch.cuda.synchronize()
    assert out.shape == (5, 6) and (out == 0).all()


def test_quantised_real_operands_config1():
    # config 1 end to end through the two calls: quantise (RNE, no rotation), then GEMM
    x = synth.normal(256, 512, 1.0, 0, synth.STREAM_X)
    w = synth.normal(512, 512, 0.02, 0, synth.STREAM_W)
    xq, xs = mx.mxfp4_quantize(x.to("cuda:0"))
    wq, ws = mx.mxfp4_quantize(w.to("cuda:0"))
    y = mx.mxfp4_gemm(xq, xs, wq, ws, out_dtype=mx.OUT_FP32)
    torch.cuda.synchronize()
    want, absum = oracle.linear_fwd(synth.as_u16(x), synth.as_u16(w))
    assert y.shape == (256, 512)
    assert_close(y.cpu().numpy(), want, absum)


def take_rows(op, rows):
    q, s_ = op
    return np.ascontiguousarray(q[rows]), np.ascontiguousarray(s_[rows])


def structured_check(out, a, b, rng, fmts=(0, 0), n_lines=64, tile=256, patch=16, close=None):
    """Parity of a large GEMM output `out` (numpy [Ra][Rb]) = A B^T on complete K-sums the oracle can afford:
    a patch x patch block at a random place inside EVERY tile x tile output tile (one random row offset per tile
    row, one random column offset per tile column: the patches are the cross product, one oracle GEMM), n_lines
    whole rows and n_lines whole columns (first and last included).  a, b: (q, s) of the operands."""
    close = close or assert_close
    Ra, Rb = out.shape

    def offsets(R):
        idx = []
        for t0 in range(0, R, tile):
            span = min(tile, R - t0)
            o = t0 + int(rng.integers(0, max(span - patch, 0) + 1))
            idx += list(range(o, min(o + patch, R)))
        return np.array(idx, dtype=np.int64)

    def gemm(x, y):
        return oracle.gemm_fmt(x[0], x[1], fmts[0], y[0], y[1], fmts[1])

    pr, pc = offsets(Ra), offsets(Rb)
    want, absum = gemm(take_rows(a, pr), take_rows(b, pc))
    close(out[np.ix_(pr, pc)], want, absum)
    rows = np.unique(np.concatenate([rng.integers(0, Ra, n_lines - 2), [0, Ra - 1]]))
    want, absum = gemm(take_rows(a, rows), b)
    close(out[rows], want, absum)
    cols = np.unique(np.concatenate([rng.integers(0, Rb, n_lines - 2), [0, Rb - 1]]))
    want, absum = gemm(a, take_rows(b, cols))
    close(out[:, cols], want, absum)


def close_bf16(got, want, absum):
    assert (np.abs(got - want) <= 1e-5 * absum + 2.0**-8 * np.abs(want)).all()


@pytest.mark.parametrize("C", [1024, 1280, 2304])
def test_many_tiles_per_workgroup_whole_output(C):
    # 17 x 17 = 289 tiles of 256 x 256 (more than one per CU, not a multiple of 8): tiles hand over inside a
    # workgroup; 4, 5 and 9 K-stages of 256 (with an odd count the stage buffers swap roles from one tile of a
    # workgroup to the next).  Every element of the output is compared, fp32 and bf16.
    Ra = Rb = 256 * 17
    assert_runs_on("tail", Ra, Rb, C)
    rng = np.random.default_rng(5)
    aq, as_ = rand_operand(rng, Ra, C)
    bq, bs = rand_operand(rng, Rb, C)
    want, absum = oracle.gemm(aq, as_, bq, bs)
    ga, gas, gb, gbs = gpu(aq), gpu(as_), gpu(bq), gpu(bs)
    f32 = mx.mxfp4_gemm(ga, gas, gb, gbs, out_dtype=mx.OUT_FP32)
    b16 = mx.mxfp4_gemm(ga, gas, gb, gbs, out_dtype=mx.OUT_BF16)
    acc = f32.clone()
    mx.mxfp4_gemm(ga, gas, gb, gbs, out=acc, out_dtype=mx.OUT_FP32, accumulate=True)
    torch.cuda.synchronize()
    assert_close(f32.cpu().numpy(), want, absum)
    assert torch.equal(b16, f32.to(torch.bfloat16))   # bf16 output = RNE of the fp32 output, everywhere
    assert torch.equal(acc, f32 + f32)                # the accumulating epilogue, everywhere


@pytest.mark.parametrize("shape", [(256 * 17, 128 * 17, 1280), (256 * 9, 128 * 35, 1024), (1024, 4096, 2048),
                                   (8192, 1024, 1024)])
def test_narrow_tiles_whole_output(shape):
    # outputs whose column count is a whole number of 128s but not of 256s, or that have fewer 256 x 256 tiles than
    # the chip has compute units, run on 256 x 128 tiles; with 289 and 315 of them a workgroup hands over from tile
    # to tile (odd and even numbers of K stages).  Every element, fp32, bf16 and accumulating.
    Ra, Rb, C = shape
    assert_runs_on("narrow", Ra, Rb, C)
    assert_runs_on("narrow", Ra, Rb, C, out_dtype=mx.OUT_FP32, ld_out=Rb + 8)
    rng = np.random.default_rng(Ra + Rb + C)
    aq, as_ = rand_operand(rng, Ra, C)
    bq, bs = rand_operand(rng, Rb, C)
    want, absum = oracle.gemm(aq, as_, bq, bs)
    ga, gas, gb, gbs = gpu(aq), gpu(as_), gpu(bq), gpu(bs)
    canvas = torch.full((Ra + 1, Rb + 8), 7.0, dtype=torch.float32, device="cuda:0")
    mx.mxfp4_gemm(ga, gas, gb, gbs, out=canvas[:Ra, :Rb], out_dtype=mx.OUT_FP32)
    b16 = mx.mxfp4_gemm(ga, gas, gb, gbs, out_dtype=mx.OUT_BF16)
    torch.cuda.synchronize()
    c = canvas.cpu().numpy()
    assert_close(c[:Ra, :Rb], want, absum)
    assert np.all(c[:Ra, Rb:] == 7.0) and np.all(c[Ra] == 7.0)          # nothing written outside
    f32 = canvas[:Ra, :Rb].clone()
    assert torch.equal(b16, f32.to(torch.bfloat16))
    mx.mxfp4_gemm(ga, gas, gb, gbs, out=canvas[:Ra, :Rb], out_dtype=mx.OUT_FP32, accumulate=True)
    torch.cuda.synchronize()
    assert torch.equal(canvas[:Ra, :Rb], f32 + f32)


@pytest.mark.parametrize("shape", [(6144, 4096, 2048), (256 * 40, 256 * 8, 1024), (4096, 14336, 1024)])
def test_part_filled_last_round_runs_on_narrow_tiles(shape):
    # 384, 320 and 896 tiles of 256 x 256 on 256 compute units: the whole rounds run on 256 x 256 tiles, the rest in
    # halves on 256 x 128 tiles in the same launch (896 tiles: the cut after 768 falls inside a row of 56 tiles);
    # every element of the output against the oracle, also when the product is added to the output
    Ra, Rb, C = shape
    assert_runs_on("tail", Ra, Rb, C)
    rng = np.random.default_rng(Ra * 3 + Rb + C)
    aq, as_ = rand_operand(rng, Ra, C)
    bq, bs = rand_operand(rng, Rb, C)
    want, absum = oracle.gemm(aq, as_, bq, bs)
    f32 = run_gemm(aq, as_, bq, bs, out_dtype=mx.OUT_FP32)
    b16 = run_gemm(aq, as_, bq, bs, out_dtype=mx.OUT_BF16)
    assert_close(f32.cpu().numpy(), want, absum)
    assert torch.equal(b16, f32.to(torch.bfloat16))
    acc = torch.full((Ra, Rb), 0.25, dtype=torch.float32, device="cuda:0")
    run_gemm(aq, as_, bq, bs, out=acc, out_dtype=mx.OUT_FP32, accumulate=True)
    assert torch.equal(acc, f32 + 0.25)


def test_config2_shape_every_tile():
    # 8192 x 6144 x 4096 (fused QKV Fprop) through the two single-operation calls: complete K-sums at a patch
    # inside every output tile, whole rows and whole columns (tests/test_gpu_configs.py compares the whole output)
    x = synth.normal(8192, 4096, 1.0, 0, synth.STREAM_X)
    w = synth.normal(6144, 4096, 0.02, 0, synth.STREAM_W)
    xq, xs = mx.mxfp4_quantize(x.to("cuda:0"), hadamard=mx.HAD_DET)
    wq, ws = mx.mxfp4_quantize(w.to("cuda:0"), hadamard=mx.HAD_DET)
    y = mx.mxfp4_gemm(xq, xs, wq, ws, out_dtype=mx.OUT_FP32)
    torch.cuda.synchronize()
    structured_check(y.cpu().numpy(), (xq.cpu().numpy(), xs.cpu().numpy()), (wq.cpu().numpy(), ws.cpu().numpy()),
                     np.random.default_rng(0))


@pytest.mark.parametrize("shapes,acc", [
    (((4096, 2048, 4096), (4096, 2048, 4096)), False),   # 128 + 128 tiles, equal work: side by side, 128 CUs each
    (((4096, 4096, 1024), (2048, 4096, 1024)), True),    # 256 + 128 tiles: split 21 : 11 per XCD, second accumulating
    (((512, 256, 1024), (96, 160, 224)), False),         # too few tiles / ragged: both on the ragged-shape kernel
    (((8192, 1024, 1024), (1024, 1024, 8192)), True),    # one after the other
    (((300, 520, 1024), (0, 64, 64)), False),            # the second product empty
])
def test_gemm_pair_equals_the_two_separate_calls(shapes, acc):
    # two independent products (App. C.2, C.3) in one call: bit for bit the results of two mxfp4_gemm calls, and
    # the first of them against the oracle
    kinds = {4096: mx.PAIR_SIDE_BY_SIDE, 512: mx.PAIR_EDGE, 8192: mx.PAIR_APART, 300: mx.PAIR_APART}
    assert mx.mxfp4_gemm_pair_route(*shapes, accumulate1=acc)[0] == kinds[shapes[0][0]]
    rng = np.random.default_rng(sum(shapes[0]) + sum(shapes[1]))
    ops = []
    for Ra, Rb, C in shapes:
        ops.append(tuple(gpu(t) for t in rand_operand(rng, Ra, C) + rand_operand(rng, Rb, C)))
    (a0q, a0s, b0q, b0s), (a1q, a1s, b1q, b1s) = ops
    base = torch.full((shapes[1][0], shapes[1][1]), 0.5, dtype=torch.float32, device="cuda:0")
    want0 = mx.mxfp4_gemm(a0q, a0s, b0q, b0s, out_dtype=mx.OUT_BF16)
    want1 = mx.mxfp4_gemm(a1q, a1s, b1q, b1s, out=base.clone(), out_dtype=mx.OUT_FP32, accumulate=acc)
    out0 = torch.empty_like(want0)
    out1 = base.clone()
    mx.mxfp4_gemm_pair((a0q, a0s), (b0q, b0s), out0, (a1q, a1s), (b1q, b1s), out1, accumulate1=acc)
    torch.cuda.synchronize()
    assert torch.equal(out0, want0) and torch.equal(out1, want1)
    ref, absum = oracle.gemm(*(t.cpu().numpy() for t in ops[0]))
    close_bf16(out0.float().cpu().numpy(), ref, absum)


@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
@pytest.mark.parametrize("shape,kernel4,kernel8", [
    ((512, 768, 1024), "64x64", "64x64"), ((512, 640, 1024), "64x64", "64x64"), ((768, 2560, 1024), "64x64", "128x64"),
    ((2048, 2560, 1024), "narrow", "128x256"), ((4096, 2176, 1280), "narrow", "moved back"),
    ((4096, 4096, 1024), "wide", "wide"), ((4352, 4352, 1024), "tail", "wide")])
def test_every_output_variant_of_the_tiled_kernels_agrees_with_the_fp32_result(shape, kernel4, kernel8, fmt):
    # each kernel's epilogues, and a strided output: the bf16 output is the rounding of the fp32 output, and the
    # accumulating call adds the fp32 output to what the buffer held, bit for bit
    Ra, Rb, C = shape
    for dt, acc in ((mx.OUT_FP32, False), (mx.OUT_BF16, False), (mx.OUT_FP32, True)):
        assert_runs_on(kernel8 if fmt else kernel4, Ra, Rb, C, fmt, out_dtype=dt, accumulate=acc)
    rng = np.random.default_rng(Ra + Rb + fmt)
    if fmt == mx.FMT_E2M1:
        a, b = rand_operand(rng, Ra, C), rand_operand(rng, Rb, C)
    else:
        a = (rng.integers(0, 120, size=(Ra, C), dtype=np.uint8), rng.integers(118, 132, size=(Ra, C // 32), dtype=np.uint8))
        b = (rng.integers(0, 120, size=(Rb, C), dtype=np.uint8), rng.integers(118, 132, size=(Rb, C // 32), dtype=np.uint8))
    ops = [gpu(t) for t in a + b]
    kw = dict(a_format=fmt, b_format=fmt)
    f32 = mx.mxfp4_gemm(*ops, out_dtype=mx.OUT_FP32, **kw)
    b16 = mx.mxfp4_gemm(*ops, out_dtype=mx.OUT_BF16, **kw)
    big = torch.full((Ra, Rb + 64), 0.375, dtype=torch.float32, device="cuda:0")
    mx.mxfp4_gemm(*ops, out=big[:, :Rb], out_dtype=mx.OUT_FP32, accumulate=True, **kw)
    torch.cuda.synchronize()
    assert torch.isfinite(f32).all()
    assert torch.equal(b16, f32.to(torch.bfloat16))
    assert torch.equal(big[:, :Rb], f32 + 0.375) and bool((big[:, Rb:] == 0.375).all())


@pytest.mark.parametrize("shapes,kind", [
    (((4096, 4096, 1024), (2048, 4096, 2048)), mx.PAIR_SIDE_BY_SIDE),   # 256 and 128 tiles, equal work: 128 compute units each
    (((2048, 4096, 1024), (4096, 2048, 1280)), mx.PAIR_APART)])         # 128 tiles each, too few for one of the shares
@pytest.mark.parametrize("dt0,dt1,acc1", [(mx.OUT_BF16, mx.OUT_BF16, False), (mx.OUT_BF16, mx.OUT_FP32, False),
                                          (mx.OUT_BF16, mx.OUT_FP32, True), (mx.OUT_FP32, mx.OUT_BF16, False),
                                          (mx.OUT_FP32, mx.OUT_FP32, False), (mx.OUT_FP32, mx.OUT_FP32, True)])
def test_every_output_variant_of_the_side_by_side_launch(dt0, dt1, acc1, shapes, kind):
    # every combination of output types
    assert mx.mxfp4_gemm_pair_route(*shapes, out_dtypes=(dt0, dt1), accumulate1=acc1)[0] == kind
    rng = np.random.default_rng(dt0 * 4 + dt1 * 2 + acc1)
    ops = [tuple(gpu(t) for t in rand_operand(rng, Ra, C) + rand_operand(rng, Rb, C)) for Ra, Rb, C in shapes]
    (a0q, a0s, b0q, b0s), (a1q, a1s, b1q, b1s) = ops
    t = lambda d: torch.float32 if d == mx.OUT_FP32 else torch.bfloat16
    base1 = torch.full((shapes[1][0], shapes[1][1]), 0.5, dtype=t(dt1), device="cuda:0")
    want0 = mx.mxfp4_gemm(a0q, a0s, b0q, b0s, out_dtype=dt0)
    want1 = mx.mxfp4_gemm(a1q, a1s, b1q, b1s, out=base1.clone(), out_dtype=dt1, accumulate=acc1)
    out0, out1 = torch.empty_like(want0), base1.clone()
    mx.mxfp4_gemm_pair((a0q, a0s), (b0q, b0s), out0, (a1q, a1s), (b1q, b1s), out1, accumulate1=acc1)
    torch.cuda.synchronize()
    assert torch.equal(out0, want0) and torch.equal(out1, want1)


def test_short_mxfp4_products_on_the_any_shape_kernel_equal_the_ragged_shape_kernel():
    # which of the two runs depends on the length of an output row: every remainder of 128 elements and of the tile
    # sizes up to the line between them, bit for bit
    rng = np.random.default_rng(12)
    for Ra, Rb, C in [(33, 48, 32), (64, 80, 96), (130, 112, 160), (63, 208, 288), (70, 144, 480)]:
        aq, as_ = rand_operand(rng, Ra, C, 100, 150)
        bq, bs = rand_operand(rng, Rb, C, 100, 150)
        ops = [gpu(t) for t in (aq, as_, bq, bs)]
        for dt, acc in ((mx.OUT_FP32, False), (mx.OUT_BF16, False), (mx.OUT_FP32, True)):
            canvas = {ld: torch.full((Ra, ld), 0.5, dtype=torch.float32 if dt else torch.bfloat16, device="cuda:0")
                      for ld in (Rb + 1, Rb + 12)}
            for ld, o in canvas.items():
                assert_runs_on("any" if ld % 4 else "64x64", Ra, Rb, C, ld_out=ld, out_dtype=dt, accumulate=acc)
                mx.mxfp4_gemm(*ops, out=o[:, :Rb], out_dtype=dt, accumulate=acc)
            assert torch.equal(canvas[Rb + 1][:, :Rb], canvas[Rb + 12][:, :Rb])
            assert all(bool((o[:, Rb:] == 0.5).all()) for o in canvas.values())


@pytest.mark.parametrize("fmt", [mx.FMT_E2M1, mx.FMT_E4M3])
def test_contraction_beyond_the_ragged_shape_kernels_offsets(fmt):
    # C = 2^24: the any-shape kernel; one live element in each of 96 blocks spread over the row and its end, products
    # and sums exact
    Ra, Rb, C = 3, 2, 1 << 24
    assert_runs_on("any", Ra, Rb, C, fmt, out_dtype=mx.OUT_FP32)
    blocks = np.linspace(0, C // 32 - 1, 96).astype(np.int64)
    rng = np.random.default_rng(13)
    one = {mx.FMT_E2M1: (0x2, 0xA), mx.FMT_E4M3: (0x38, 0xB8)}[fmt]     # +1, -1

    def operand(R):
        q = np.zeros((R, C // 32, 16 if fmt == mx.FMT_E2M1 else 32), dtype=np.uint8)
        v = rng.integers(0, 2, size=(R, len(blocks)))
        q[:, blocks, 0] = np.where(v, one[0], one[1])
        s = np.full((R, C // 32), 127, dtype=np.uint8)
        e = rng.integers(0, 5, size=(R, len(blocks)))
        s[:, blocks] = 127 + e
        return q.reshape(R, -1), s, np.where(v, 1.0, -1.0) * 2.0 ** e
    (aq, as_, av), (bq, bs, bv) = operand(Ra), operand(Rb)
    got = mx.mxfp4_gemm(gpu(aq), gpu(as_), gpu(bq), gpu(bs), out_dtype=mx.OUT_FP32, a_format=fmt, b_format=fmt)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), av @ bv.T)
