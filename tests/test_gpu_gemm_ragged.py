"""GPU parity of ragged GEMMs (row and column counts in no whole tiles, contraction lengths in no whole stages) around the
edges of the kernels' tiles, stages and scale batches, against the CPU oracle (exact fp64 sums; App. C.1-C.3
products).  Tolerance as in the other GEMM tests: 1e-5 * sum|a||b| for MXFP4 (fp32 sums of at most C/32 partial results,
each within 2^-24 of the running magnitude), FP8_RTOL for MXFP8 (the matrix unit drops low bits of E4M3 products)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_09825_amd as mx
from gpu_util import assert_runs_on
from test_gpu_fp8 import FP8_RTOL, rand_fp4, rand_fp8
from test_gpu_gemm import RTOL, gpu

pytestmark = pytest.mark.gpu

# 64 x 64 tiles (and, of the shorter contractions, the any-shape kernel for thin outputs or one of the two row lengths): one
# row / one tile less, whole and more; K of one block, around one stage (256 MXFP4 or 128 MXFP8 elements), around one scale
# batch (1024) and of several batches with a ragged end
SMALL = [(1, 1, 32), (63, 65, 224), (64, 64, 256), (65, 127, 288), (129, 8, 96), (24, 200, 992), (33, 72, 1024),
         (70, 66, 1056), (100, 136, 2016), (8, 24, 3232), (96, 64, 128), (96, 64, 160)]
# enough tiles for 128 x 64 and for 128 x 256 ones (rows of whole 16 bytes or not): ragged on both sides
LARGE = [(1000, 1700, 288), (1010, 1537, 1120), (2049, 1290, 2080), (2008, 3100, 736), (2001, 3075, 1056)]
# enough of everything for the 256 x 256 tiles of the tiled kernel, moved back at the edges (where rows are whole 16 bytes; the
# others, and the two smallest in MXFP8, on 128 x 256 tiles): halves of tiles only, a last round in halves, several whole tiles
# per workgroup; C in whole blocks of 32, 64, 128 and 256, odd and even stage counts; only the rows or only the contraction
# ragged
TILED = [(2300, 3000, 2080), (4200, 4104, 1056), (4900, 4904, 1120), (4352, 4352, 1408), (4300, 4352, 1280)]


def test_which_kernels_the_shapes_are_for():
    for Ra, Rb, C in SMALL:
        kernel = "any" if Ra == 1 or Rb == 8 else "64x64"
        assert_runs_on(kernel, Ra, Rb, C, ld_out=Rb + 16 - Rb % 8)
    for (Ra, Rb, C), kernel in zip(LARGE, ("64x64", "128x64", "128x64", "128x256", "128x256")):
        for fmt in (0, 1):
            assert_runs_on(kernel, Ra, Rb, C, fmt, ld_out=Rb + 3)
    for Ra, Rb, C in TILED:
        assert_runs_on("moved back", Ra, Rb, C, ld_out=Rb + 16)
        assert_runs_on("128x256", Ra, Rb, C, ld_out=Rb + 3)
    for Ra, Rb, C in [TILED[2], TILED[4]]:
        assert_runs_on("moved back", Ra, Rb, C, mx.FMT_E4M3, ld_out=Rb + 16)


@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("shape", SMALL + LARGE + TILED)
def test_every_output_once_and_nothing_outside(shape, fmt):
    Ra, Rb, C = shape
    print(f"[ragged] Ra={Ra} Rb={Rb} C={C} fmt={fmt}", flush=True)
    rng = np.random.default_rng(Ra * 13 + Rb * 7 + C + fmt)
    (aq, as_), (bq, bs) = [(rand_fp8 if fmt else rand_fp4)(rng, R, C) for R in (Ra, Rb)]
    want, absum = oracle.gemm_fmt(aq, as_, fmt, bq, bs, fmt)
    args = [gpu(t) for t in (aq, as_, bq, bs)]
    fmts = dict(a_format=fmt, b_format=fmt)
    results = []
    for ld in (Rb + 8 - Rb % 8 + 8, Rb + 3):   # rows of whole 16 bytes, and of any length
        canvas = torch.full((Ra + 1, ld), 7.0, dtype=torch.float32, device="cuda:0")
        mx.mxfp4_gemm(*args, out=canvas[:Ra, :Rb], out_dtype=mx.OUT_FP32, **fmts)
        torch.cuda.synchronize()
        c = canvas.cpu().numpy()
        assert np.all(np.abs(c[:Ra, :Rb] - want) <= (FP8_RTOL if fmt else RTOL) * absum)
        assert np.all(c[:Ra, Rb:] == 7.0) and np.all(c[Ra] == 7.0)
        mx.mxfp4_gemm(*args, out=canvas[:Ra, :Rb], out_dtype=mx.OUT_FP32, accumulate=True, **fmts)
        first = torch.from_numpy(c[:Ra, :Rb].copy())
        assert torch.equal(canvas[:Ra, :Rb].cpu(), first + first)
        half = torch.full((Ra + 1, ld), 7.0, dtype=torch.bfloat16, device="cuda:0")
        mx.mxfp4_gemm(*args, out=half[:Ra, :Rb], out_dtype=mx.OUT_BF16, **fmts)
        h = half.cpu()
        assert torch.equal(h[:Ra, :Rb], first.to(torch.bfloat16))
        assert bool((h[:Ra, Rb:] == 7.0).all()) and bool((h[Ra] == 7.0).all())
        results.append(first)
    assert torch.equal(results[0], results[1])


@pytest.mark.parametrize("shape", [(70, 66, 1056), (2001, 3075, 1056), (4200, 4104, 1056)])
def test_scale_byte_ff_in_the_ragged_last_block_marks_its_row_only(shape):
    Ra, Rb, C = shape
    rng = np.random.default_rng(5)
    (aq, as_), (bq, bs) = rand_fp4(rng, Ra, C), rand_fp4(rng, Rb, C)
    as_[3, C // 32 - 1] = 0xFF
    bs[Rb - 1, 0] = 0xFF
    got = mx.mxfp4_gemm(gpu(aq), gpu(as_), gpu(bq), gpu(bs), out_dtype=mx.OUT_FP32).cpu().numpy()
    nan = np.isnan(got)
    assert nan[3].all() and nan[:, Rb - 1].all() and nan.sum() == Ra + Rb - 1
