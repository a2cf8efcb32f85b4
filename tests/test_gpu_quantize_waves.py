"""GPU tests: the column-wise quantisers' workgroups of eight waves, which large tensors alone get: both axes without a rotation, two tensors of which
one is beyond the last-level cache, MXFP8 beyond 2^25 elements, MXFP8 beside MXFP4.  Ragged everywhere; byte for byte the row-wise kernels on
the transposed tensor, or (32 x 32 regions) the same calls on parts of it that get four waves."""
import pytest
import torch

import paper_2605_09825_amd as mx

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def tensor(rows, cols, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.empty((rows, cols), dtype=torch.bfloat16, device=DEV)
    for r in range(0, rows, 2048):  # (in pieces: a tenth of the memory)
        x[r:r + 2048] = torch.randn((min(2048, rows - r), cols), generator=g, device=DEV).to(torch.bfloat16)
    return x


def rowwise(x, had, fp8=False, rnd=mx.RNE, seed=0):
    return mx.mxfp4_quantize_fp8(x, mx.AXIS_LAST, had, seed) if fp8 else mx.mxfp4_quantize(x, mx.AXIS_LAST, had, rnd, seed)


def regions_in_parts(x, had):
    """(q, s) of the rows of x under 32 x 32 regions, a few rows at a time (four waves)."""
    parts = [mx.mxfp4_quantize_2d(x[r:r + 512], had, want_first=False)[:2] for r in range(0, x.shape[0], 512)]
    return tuple(torch.cat(p) for p in zip(*parts))


def same(got, want):
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("cols", [6176, 6304])
def test_both_axes_without_a_rotation(cols):
    x = tensor(8224, cols, 1)  # 33 x 49, 33 x 50 tiles of eight
    ql, sl, qf, sf = mx.mxfp4_quantize_dual(x)
    same((ql, sl), rowwise(x, mx.HAD_NONE))
    same((qf, sf), rowwise(x.T.contiguous(), mx.HAD_NONE))


@pytest.mark.parametrize("axes", [(True, True), (False, True), (True, False)])
def test_regions_without_a_rotation(axes):
    x = tensor(8224, 6176, 2)
    ql, sl, qf, sf = mx.mxfp4_quantize_2d(x, want_last=axes[0], want_first=axes[1])
    if axes[0]:
        same((ql, sl), regions_in_parts(x, mx.HAD_NONE))
    if axes[1]:
        same((qf, sf), regions_in_parts(x.T.contiguous(), mx.HAD_NONE))


# X beyond the last-level cache, W not
@pytest.mark.parametrize("had", [mx.HAD_NONE, mx.HAD_DET])
@pytest.mark.parametrize("geometry", [mx.GEOM_1D, mx.GEOM_2D])
def test_two_tensors_one_beyond_the_cache(geometry, had):
    M, N, K = 16416, 96, 8224
    x, w = tensor(M, K, 3), tensor(N, K, 4)
    cfg = mx.make_cfg(had, mx.RNE, 0, geometry=geometry)
    _, ws, saved = mx.mxfp4_linear_fwd_save(x, w, cfg)
    of = lambda buf, at, R, C: (buf[at[0]:at[0] + R * C // 2].view(R, C // 2), buf[at[1]:at[1] + R * C // 32].view(R, C // 32))
    fw, sv = mx.mxfp4_linear_workspace_layout(M, N, K, False, cfg), mx.mxfp4_linear_saved_layout(M, N, K, cfg)
    want = (lambda t: regions_in_parts(t, had)) if geometry == mx.GEOM_2D else (lambda t: rowwise(t, had))
    same(of(ws, fw[:2], M, K), want(x))
    same(of(ws, fw[2:4], N, K), want(w))
    same(of(saved, sv[:2], K, N), want(w.T.contiguous()))
    same(of(saved, sv[2:], K, M), want(x.T.contiguous()))


@pytest.mark.parametrize("cols", [8290, 8224])
def test_mxfp8(cols):
    x = tensor(8224, cols, 5)
    xt = x.T.contiguous()
    same(mx.mxfp4_quantize_fp8(x, mx.AXIS_FIRST, mx.HAD_DET), rowwise(xt, mx.HAD_DET, fp8=True))
    if cols % 32 == 0:
        ql, sl, qf, sf = mx.mxfp4_quantize_fp8_dual(x, mx.HAD_DET)
        same((ql, sl), rowwise(x, mx.HAD_DET, fp8=True))
        same((qf, sf), rowwise(xt, mx.HAD_DET, fp8=True))


@pytest.mark.parametrize("had,rnd", [(mx.HAD_NONE, mx.RNE), (mx.HAD_DET, mx.RNE), (mx.HAD_RANDSIGN, mx.SR)])
def test_mxfp8_beside_mxfp4(had, rnd):
    M, N, K, seed = 8224, 32, 8224, 11
    x, w = tensor(M, K, 6), tensor(N, K, 7)
    cfg = mx.make_cfg(had, rnd, seed, dgrad_format=mx.FMT_E4M3, wgrad_format=mx.FMT_E4M3)
    _, ws, saved = mx.mxfp4_linear_fwd_save(x, w, cfg)
    fw, sv = mx.mxfp4_linear_workspace_layout(M, N, K, False, cfg), mx.mxfp4_linear_saved_layout(M, N, K, cfg)
    q, s = rowwise(x, had, rnd=rnd, seed=seed)
    assert torch.equal(ws[fw[0]:fw[0] + q.numel()], q.flatten()) and torch.equal(ws[fw[1]:fw[1] + s.numel()], s.flatten())
    q, s = rowwise(x.T.contiguous(), mx.HAD_NONE, fp8=True)  # (MXFP8 operands are neither rotated nor rounded stochastically)
    assert torch.equal(saved[sv[2]:sv[2] + q.numel()], q.flatten()) and torch.equal(saved[sv[3]:sv[3] + s.numel()], s.flatten())
