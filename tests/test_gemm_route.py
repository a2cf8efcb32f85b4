"""CPU-only checks of the rule that decides which kernel a product, or a pair of products, runs on (256 compute units; no
device is touched).  GPU tests that are about one kernel ask the same functions, so that they cannot leave it unnoticed."""
import ctypes

import paper_2605_09825_amd as mx

route, pair = mx.mxfp4_gemm_route, mx.mxfp4_gemm_pair_route
FP8 = dict(a_format=mx.FMT_E4M3, b_format=mx.FMT_E4M3)


def test_whole_tiles_that_fill_the_chip_run_as_planned():
    for shape in [(8192, 6144, 4096), (6144, 4096, 8192), (8192, 1024, 4096), (4096, 14336, 16384)]:
        assert route(*shape) == mx.ROUTE_BLOCKS
        assert route(*shape, out_dtype=mx.OUT_FP32, accumulate=True) == mx.ROUTE_BLOCKS
    assert route(8192, 6144, 4096, **FP8) == mx.ROUTE_BLOCKS


def test_large_ragged_products_leave_the_plan():
    # (the plan of the first is a tiled interior and a strip, of the second one block on the kernels for other shapes)
    assert len(mx.mxfp4_gemm_plan(4010, 6144, 4096)) == 2
    for shape in [(4010, 6144, 4096), (8192, 6144, 4064), (8192, 28640, 4064)]:
        assert route(*shape) == mx.ROUTE_RAGGED_TILED
    assert route(8192, 6144, 4064, **FP8) == mx.ROUTE_RAGGED_TILED
    assert route(8192, 6144, 4064, ld_out=6148) == mx.ROUTE_EDGE_256    # rows of the output not 16-byte aligned


def test_whole_128s_of_columns():
    for shape in [(14848, 3456, 1024), (7168, 10368, 1024), (6144, 5760, 1792)]:
        assert route(*shape) == mx.ROUTE_BLOCKS and mx.mxfp4_gemm_plan(*shape)[0][0] == mx.GEMM_TILED_128
        assert route(*shape, out_dtype=mx.OUT_FP32) == mx.ROUTE_RAGGED_TILED
    assert route(6144, 5760, 2048) == mx.ROUTE_RAGGED_TILED
    assert route(14592, 3448, 1056) == mx.ROUTE_RAGGED_TILED            # no whole tiles of either width


def test_products_too_small_for_whole_tiles():
    assert route(24, 6144, 4096) == mx.ROUTE_EDGE_64
    assert route(2080, 4320, 1440) == mx.ROUTE_EDGE_128
    assert route(300, 520, 1024) == mx.ROUTE_EDGE_64
    assert route(512, 4096, 4096, **FP8) == mx.ROUTE_EDGE_128
    assert route(0, 16, 32) == route(16, 0, 32) == mx.ROUTE_NONE
    for f in [dict(a_format=mx.FMT_E4M3), dict(b_format=mx.FMT_E4M3)]:  # operands of different formats
        assert route(24, 6144, 4096, **f) == route(8192, 6144, 4096, **f) == mx.ROUTE_ANY_SHAPE


def test_short_products_stay_on_the_any_shape_kernel():
    ANY = mx.ROUTE_ANY_SHAPE
    fp32 = dict(out_dtype=mx.OUT_FP32)
    # rows of the output in no whole 4s: below 256 bytes of codes per row, at most a tile of 64 x 64 per compute unit
    for C, f in [(480, {}), (224, FP8)]:
        assert route(1000, 1000, C, ld_out=1003, **f) == ANY
        assert route(1000, 1000, C + 32, ld_out=1003, **f) == mx.ROUTE_EDGE_64
        assert route(1000, 1000, C, ld_out=1003, out_dtype=mx.OUT_FP32, accumulate=True, **f) == ANY
        assert route(1000, 1000, C, **f) == mx.ROUTE_EDGE_64
    assert route(1000, 1000, 256, ld_out=1003) == mx.ROUTE_EDGE_64 and route(32, 1000, 256, ld_out=1003) == ANY
    assert route(10736, 88, 128, ld_out=91) == ANY and route(10736, 88, 160, ld_out=91) != ANY       # 336 tiles
    assert route(64 * 385, 30, 128, ld_out=31) != ANY
    # few rows or columns
    assert route(32, 1000, 256) == route(1000, 32, 256) == route(32, 1000, 256, **fp32) == ANY
    assert route(33, 1000, 256) == route(32, 1000, 256, accumulate=True, **fp32) == mx.ROUTE_EDGE_64
    assert route(1000, 16, 480, accumulate=True, **fp32) == route(16, 1000, 352, **FP8) == ANY
    assert route(1000, 16, 512) == route(1000, 17, 256, **FP8) == route(16, 1000, 384, **FP8) == mx.ROUTE_EDGE_64
    assert route(64 * 384, 16, 32) == ANY and route(64 * 384 + 1, 16, 32) != ANY
    assert route(1000, 20, 256, accumulate=True, **fp32) == mx.ROUTE_EDGE_64
    # one K-step, columns in no whole 16s
    assert route(200, 200, 128) == ANY and route(200, 208, 128) == route(200, 200, 160) == mx.ROUTE_EDGE_64
    # a pair is one launch all the same
    assert pair((200, 200, 128), (32, 64, 128))[0] == mx.PAIR_EDGE


def test_short_rows_take_small_tiles_while_the_chip_holds_them():
    for C, f in [(1024, {}), (512, FP8)]:
        assert route(64 * 64, 64 * 8, C, **f) == mx.ROUTE_EDGE_64          # 512 tiles of 64 x 64, 512 bytes per row
        assert route(64 * 64, 64 * 8, C + 32, **f) == mx.ROUTE_EDGE_128
        assert route(64 * 64 + 1, 64 * 8, C, **f) != mx.ROUTE_EDGE_64
    assert pair((64 * 32, 64 * 8, 1024), (64 * 32, 64 * 8, 512)) == (mx.PAIR_EDGE, 0, 0, 0)
    assert pair((64 * 32, 64 * 8, 1056), (64 * 32, 64 * 8, 512)) == (mx.PAIR_EDGE, 0, 1, 0)


def test_pairs():
    dgrad_wgrad = lambda M, N, K: ((M, K, N), (N, K, M))
    assert pair(*dgrad_wgrad(8192, 6144, 4096)) == (mx.PAIR_SIDE_BY_SIDE, 0, 16, 0)
    # few narrow tiles of the one beside many wide ones of the other: of Wgrad, of Dgrad
    assert pair(*dgrad_wgrad(8192, 1024, 4096)) == (mx.PAIR_NARROW_BESIDE_WIDE, 1, 16, 128)
    assert pair(*dgrad_wgrad(1024, 4096, 4096))[:3] == (mx.PAIR_NARROW_BESIDE_WIDE, 0, 16)
    assert pair(*dgrad_wgrad(2080, 4320, 1440))[0] == mx.PAIR_EDGE
    assert pair((64, 64, 32), (64, 64, 4096))[:2] == (mx.PAIR_EDGE, 1)  # the longer contraction starts first
    assert pair((300, 520, 1024), (0, 64, 64))[0] == mx.PAIR_APART     # one of them empty
    # a smaller chip: no launch that counts on 8 XCDs of 32 compute units
    assert pair(*dgrad_wgrad(8192, 6144, 4096), compute_units=128)[0] in (mx.PAIR_APART, mx.PAIR_EDGE)


def test_moved_back_pairs_but_for_narrow_outputs():
    MOVED_BACK = 3
    dgrad_wgrad = lambda M, N, K: ((M, K, N), (N, K, M))
    for layer in ((2080, 4320, 1440), (4128, 4320, 4064), (2592, 5344, 1280), (4960, 1120, 4960)):
        assert pair(*dgrad_wgrad(*layer))[::2] == (mx.PAIR_EDGE, MOVED_BACK)
    for layer in ((2496, 8704, 544), (8448, 15744, 320), (8096, 7232, 288)):  # 288 to 544 columns: up to 1.78 times the outputs in tiles
        assert pair(*dgrad_wgrad(*layer))[2] < MOVED_BACK


def test_weight_gradients_of_a_few_tokens_that_are_added_to():
    dgrad_wgrad = lambda M, N, K: ((M, K, N), (N, K, M))
    for layer in ((256, 8192, 2304), (512, 14080, 1024), (32, 8384, 2784)):
        assert pair(*dgrad_wgrad(*layer))[::2] == pair(*dgrad_wgrad(544, *layer[1:]), accumulate1=True)[::2] == (mx.PAIR_EDGE, 2)
        assert pair(*dgrad_wgrad(*layer), accumulate1=True)[::2] == (mx.PAIR_EDGE, 1)


def test_more_tiles_than_a_grid_can_hold():
    # A launch holds fewer than 2^32 threads along a dimension: 2^24 workgroups on 64 x 64 or 128 x 64 tiles, 2^23 on
    # 128 x 256 ones.  Beyond that the next larger tile, then the any-shape kernel, whose grid has two dimensions.
    assert route(64 * (2**24 - 8), 64, 32) == mx.ROUTE_EDGE_128
    assert route(720_000_000, 130, 32) == mx.ROUTE_EDGE_256             # (16.9 million tiles of 128 x 64)
    assert route(2**30 - 64, 300, 32) == mx.ROUTE_ANY_SHAPE             # (16.8 million tiles of 128 x 256)
    assert route(2**30 - 64, 300, 32, **FP8) == mx.ROUTE_ANY_SHAPE
    # a pair shares one grid: each fits, both do not
    assert pair((720_000_000, 130, 32), (64, 64, 64))[0] == mx.PAIR_EDGE
    assert pair((720_000_000, 130, 32), (720_000_000, 130, 64))[0] == mx.PAIR_APART


def test_argument_errors():
    L, r, p4 = mx.lib(), ctypes.c_int(7), (ctypes.c_int * 4)()
    ok = (16, 16, 32, 0, 0, 16, mx.OUT_FP32, 0)
    one = lambda *a, cus=256, out=ctypes.byref(r): L.mxfp4_gemm_route(*a, cus, out)
    assert one(*ok) == mx.OK
    assert one(*ok, out=None) == one(*ok, cus=0) == one(16, 16, 32, 7, *ok[4:]) == mx.EINVAL
    assert one(*ok[:6], mx.OUT_BF16, 1) == one(*ok[:6], 5, 0) == mx.EINVAL
    assert one(16, 16, 48, *ok[3:]) == one(-1, *ok[1:]) == one(*ok[:5], 8, *ok[6:]) == mx.ESHAPE
    assert one((1 << 36) + 1, *ok[1:]) == mx.ESHAPE
    half = (16, 16, 32, 0, 16, mx.OUT_FP32)
    two = lambda a, b, acc=0, cus=256, out=p4: L.mxfp4_gemm_pair_route(*a, *b, acc, cus, out)
    assert two(half, half) == mx.OK
    assert two(half, half, out=None) == two(half, half, cus=0) == two(half, half, acc=2) == mx.EINVAL
    assert two(half, (16, 16, 32, 3, 16, 1)) == two((16, 16, 32, 0, 16, 9), half) == mx.EINVAL
    assert two((16, 16, 48, 0, 16, 1), half) == two(half, (16, 16, 32, 0, 8, 1)) == mx.ESHAPE
