"""GPU parity on seeded random shapes, strides and modes: the quantiser (single- and dual-axis), the GEMM around
its tile sizes, and the linear calls, each against the oracle (bit-exact bytes; GEMM outputs within
1e-5 * sum|a||b|, App. A.1 eq. (1), App. C).  The fixed parametrisations elsewhere cover the edges by hand; this
file covers combinations nobody wrote down."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_09825_amd as mx
from paper_2605_09825_amd import synth
from test_gpu_linear import ws_slices

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("seed", [11, 12])
def test_quantiser_on_random_shapes_strides_and_modes(seed):
    rng = np.random.default_rng(seed)
    L = mx.lib()
    for it in range(30):
        axis, had, rnd = int(rng.integers(0, 2)), int(rng.integers(0, 5)), int(rng.integers(0, 2))
        qseed = int(rng.integers(0, 2**63))
        if axis == mx.AXIS_LAST:
            rows, cols, pad = int(rng.integers(1, 700)), 32 * int(rng.integers(1, 40)), 8 * int(rng.integers(0, 3))
        else:
            rows, cols, pad = 32 * int(rng.integers(1, 30)), 2 * int(rng.integers(1, 500)), 2 * int(rng.integers(0, 5))
        ld = cols + pad
        gen = (lambda: synth.normal(rows, ld, 1.0, it, synth.STREAM_X),
               lambda: synth.student_t3(rows, ld, 1e-3, it, synth.STREAM_DY),
               lambda: synth.normal_with_outlier_channels(rows, ld, it, synth.STREAM_X))[int(rng.integers(0, 3))]
        x = gen()
        print(f"[quantiser] seed={seed} it={it} axis={axis} had={had} rnd={rnd} rows={rows} cols={cols} ld={ld}",
              flush=True)
        xb, xg = synth.as_u16(x)[:, :cols], x.to(DEV)[:, :cols]
        q, s = mx.mxfp4_quantize(xg, axis, had, rnd, qseed)
        torch.cuda.synchronize()
        qo, so = oracle.quantize(xb, axis=axis, had=had, rnd=rnd, seed=qseed)
        assert np.array_equal(s.cpu().numpy(), so) and np.array_equal(q.cpu().numpy(), qo)
        if rows % 32 == 0 and cols % 32 == 0 and ld % 8 == 0:   # the same tensor through the dual-axis call
            ql = torch.empty((rows, cols // 2), dtype=torch.uint8, device=DEV)
            sl = torch.empty((rows, cols // 32), dtype=torch.uint8, device=DEV)
            qf = torch.empty((cols, rows // 2), dtype=torch.uint8, device=DEV)
            sf = torch.empty((cols, rows // 32), dtype=torch.uint8, device=DEV)
            rc = L.mxfp4_quantize_dual(xg.data_ptr(), rows, cols, ld, had, rnd, qseed, ql.data_ptr(), sl.data_ptr(),
                                       qf.data_ptr(), sf.data_ptr(), torch.cuda.current_stream().cuda_stream)
            assert rc == mx.OK
            torch.cuda.synchronize()
            for axis2, (qg, sg) in ((mx.AXIS_LAST, (ql, sl)), (mx.AXIS_FIRST, (qf, sf))):
                qo, so = oracle.quantize(xb, axis=axis2, had=had, rnd=rnd, seed=qseed)
                assert np.array_equal(sg.cpu().numpy(), so) and np.array_equal(qg.cpu().numpy(), qo)


@pytest.mark.parametrize("seed", [21, 22])
def test_gemm_on_random_shapes_around_the_tile_sizes(seed):
    rng = np.random.default_rng(seed)

    def operand(R, C):
        return (rng.integers(0, 256, size=(R, C // 2), dtype=np.uint8),
                rng.integers(112, 140, size=(R, C // 32), dtype=np.uint8))
    for it in range(16):
        kind = it % 4
        if kind == 0:    # whole tiles, any mix of 256- and 128-wide
            Ra, Rb, C = 256 * int(rng.integers(1, 8)), 128 * int(rng.integers(1, 12)), 256 * int(rng.integers(4, 12))
        elif kind == 1:  # anything
            Ra, Rb, C = int(rng.integers(1, 900)), int(rng.integers(1, 900)), 32 * int(rng.integers(1, 70))
        elif kind == 2:  # tiled interior with ragged edges
            Ra = 256 * int(rng.integers(1, 5)) + int(rng.integers(0, 200))
            Rb = 256 * int(rng.integers(1, 5)) + int(rng.integers(0, 200))
            C = 256 * int(rng.integers(4, 9))
        else:            # more tiles than compute units: several tiles per workgroup, part-filled last rounds
            Ra, Rb, C = 256 * int(rng.integers(8, 20)), 256 * int(rng.integers(8, 20)), 1024
        dt = int(rng.integers(0, 2))
        print(f"[gemm] seed={seed} it={it} Ra={Ra} Rb={Rb} C={C} out_dtype={dt}", flush=True)
        aq, as_ = operand(Ra, C)
        bq, bs = operand(Rb, C)
        out = mx.mxfp4_gemm(*(torch.from_numpy(t).to(DEV) for t in (aq, as_, bq, bs)), out_dtype=dt)
        torch.cuda.synchronize()
        want, absum = oracle.gemm(aq, as_, bq, bs)
        tol = 1e-5 * absum + (2.0**-8 * np.abs(want) if dt == mx.OUT_BF16 else 0.0)
        assert (np.abs(out.float().cpu().numpy().astype(np.float64) - want) <= tol).all()


def test_linear_calls_on_random_shapes_and_modes():
    rng = np.random.default_rng(31)
    for it in range(20):
        big = it % 5 == 0   # every fifth case is in whole tiles (too few of them for the tiled GEMM kernels)
        M = 256 * int(rng.integers(1, 6)) if big else 32 * int(rng.integers(1, 12))
        N = 256 * int(rng.integers(1, 6)) if big else 32 * int(rng.integers(1, 12))
        K = 256 * int(rng.integers(4, 8)) if big else 32 * int(rng.integers(1, 12))
        had, rnd, seed = int(rng.integers(0, 5)), int(rng.integers(0, 2)), int(rng.integers(0, 2**47))
        geom = int(rng.integers(0, 2)) if rnd == mx.RNE else mx.GEOM_1D
        print(f"[linear] it={it} M={M} N={N} K={K} had={had} rnd={rnd} geom={geom}", flush=True)
        x = synth.normal(M, K, 1.0, it, synth.STREAM_X)
        w = synth.normal(N, K, 0.02, it, synth.STREAM_W)
        dy = synth.normal(M, N, 1e-3, it, synth.STREAM_DY)
        cfg = mx.make_cfg(had, rnd, seed, y_dtype=mx.OUT_FP32, dx_dtype=mx.OUT_FP32, dw_dtype=mx.OUT_FP32,
                          geometry=geom)
        xg, wg, dyg = x.to(DEV), w.to(DEV), dy.to(DEV)
        y, ws_f = mx.mxfp4_linear_fwd(xg, wg, cfg)
        dx, dw, ws_b = mx.mxfp4_linear_bwd(dyg, xg, wg, cfg)
        y2, _, saved = mx.mxfp4_linear_fwd_save(xg, wg, cfg)
        dx2, dw2, _ = mx.mxfp4_linear_bwd_saved(dyg, saved, K, cfg)
        torch.cuda.synchronize()
        assert torch.equal(y, y2) and torch.equal(dx, dx2) and torch.equal(dw, dw2)
        xb, wb, dyb = synth.as_u16(x), synth.as_u16(w), synth.as_u16(dy)
        ops = (list(oracle.linear_fwd_operands(xb, wb, had, rnd, seed, geom)) +
               list(oracle.linear_dgrad_operands(dyb, wb, had, rnd, seed, geom)) +
               list(oracle.linear_wgrad_operands(dyb, xb, had, rnd, seed, geom)))
        got = ws_slices(ws_f, M, N, K, False) + ws_slices(ws_b, M, N, K, True)
        for k, ((q, s), (qo, so)) in enumerate(zip(got, ops)):
            assert np.array_equal(s, so) and np.array_equal(q, qo), f"operand {k}"
        for out, (a, b) in ((y, ops[0:2]), (dx, ops[2:4]), (dw, ops[4:6])):
            want, absum = oracle.gemm(a[0], a[1], b[0], b[1])
            assert (np.abs(out.cpu().numpy().astype(np.float64) - want) <= 1e-5 * absum).all()
