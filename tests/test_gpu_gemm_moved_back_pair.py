"""GPU tests: Dgrad and Wgrad of layers with ragged widths in one launch on moved-back tiles, in every combination of tile shapes, output types and
accumulation: bit for bit the results of the separate calls, and nothing written outside."""
import numpy as np
import pytest
import torch

import paper_2605_09825_amd as mx
from test_gpu_fp8 import rand_fp4
from test_gpu_gemm import gpu

pytestmark = pytest.mark.gpu

MOVED_BACK = 3
# M, N, K of the layer; which of the two products (Dgrad, Wgrad) are on 256 x 128 tiles
LAYERS = [((2080, 4320, 1440), (True, False)), ((3040, 2720, 2016), (False, False)), ((4960, 1120, 4960), (False, False)),
          ((6400, 2048, 1120), (False, True)), ((1504, 1504, 8160), (True, True))]


def test_tile_shapes():
    seen = set()
    for (M, N, K), narrow in LAYERS:
        kind, first, n, split = mx.mxfp4_gemm_pair_route((M, K, N), (N, K, M))
        assert (kind, first, n) == (mx.PAIR_EDGE, 0, MOVED_BACK) and 0 < split % 32 < 32
        assert (bool(split & 32), bool(split & 64)) == narrow
        seen.add(narrow)
    assert len(seen) == 4


@pytest.mark.parametrize("dx_dtype,accumulate", [(mx.OUT_BF16, False), (mx.OUT_BF16, True), (mx.OUT_FP32, False), (mx.OUT_FP32, True)])
@pytest.mark.parametrize("layer", [l for l, _ in LAYERS])
def test_equals_the_single_calls(layer, dx_dtype, accumulate):
    M, N, K = layer
    shapes = ((M, K, N), (N, K, M))
    assert mx.mxfp4_gemm_pair_route(*shapes, out_dtypes=(dx_dtype, mx.OUT_FP32), accumulate1=accumulate)[2] == MOVED_BACK
    rng = np.random.default_rng(M + N + K)
    ops = [[tuple(gpu(t) for t in rand_fp4(rng, R, C)) for R in (Ra, Rb)] for Ra, Rb, C in shapes]
    dtype = torch.float32 if dx_dtype == mx.OUT_FP32 else torch.bfloat16
    canvas0 = torch.full((M + 1, K), 7.0, dtype=dtype, device="cuda:0")
    canvas1 = torch.full((N + 1, K), 0.5, dtype=torch.float32, device="cuda:0")
    mx.mxfp4_gemm_pair(*ops[0], canvas0[:M], *ops[1], canvas1[:N], accumulate1=accumulate)
    want0 = mx.mxfp4_gemm(*ops[0][0], *ops[0][1], out_dtype=dx_dtype)
    want1 = mx.mxfp4_gemm(*ops[1][0], *ops[1][1], out=torch.full((N, K), 0.5, device="cuda:0"), accumulate=accumulate)
    assert torch.equal(canvas0[:M], want0) and torch.equal(canvas1[:N], want1)
    assert bool((canvas0[M] == 7.0).all()) and bool((canvas1[N] == 0.5).all())
