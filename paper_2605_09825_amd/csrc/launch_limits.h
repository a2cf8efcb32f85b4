// Host rules about launch grids, free of HIP types.
#pragma once
#include <stdint.h>

namespace mxfp4 {

// HIP refuses a launch of 2^32 or more threads along one dimension of the grid.
constexpr bool grid_fits(int64_t groups, int threads) { return groups < (int64_t(1) << 32) / threads; }

// MI355X Infinity Cache: the quantisers store the codes of a tensor larger than it past the caches
constexpr int64_t LLC_BYTES = int64_t(256) << 20;
constexpr bool beyond_llc(int64_t rows, int64_t cols) { return rows * cols * 2 > LLC_BYTES; }

// Workgroups of the MXFP4 quantisers: row-wise 256 threads for 256 blocks, column-wise 512 threads for 128 columns x 8
// block rows (or 256 threads for 128 columns x 4 block rows: twice the workgroups of the same number of threads in all).
constexpr int ROWS_THREADS = 256, COLS_THREADS = 512;
constexpr int64_t rows_groups(int64_t rows, int64_t cols) { return (rows * (cols / 32) + 255) / 256; }
constexpr int64_t cols_groups(int64_t rows, int64_t cols) { return ((cols + 127) / 128) * ((rows / 32 + 7) / 8); }

// Waves, and so blocks of 32 rows, per workgroup of the MXFP4 column-wise kernels, for one tensor or two in a launch.  Four where the vector
// instructions or the chain through one workgroup are what bounds (stochastic rounding, rotations of both axes, few tiles): the halves of a tile
// of eight then run on compute units of their own, and wait for each other less.  Eight, whose output rows get whole 128-byte lines, where memory
// does.  Time with four over time with eight, rounding to nearest (us with eight / four), of both axes with the GEMM behind them:
//   * one axis: from 512 tiles of eight on 1.0 to 1.15 (8192 x 14336 47 / 51), below 0.87 to 1.01 (2080 x 1440 5.2 / 4.6);
//   * both axes, no rotation: from 1536 tiles on 1.02 to 1.06 (X and W of M x N x K 4096 x 4096 x 14336 175 / 180), 0.98 to 1.0 from 192 on,
//     0.93 below 128; 32 x 32 regions alike (173 / 181);
//   * both axes, rotated: 0.9 below 128 tiles, 0.96 below 1536, 1.0 beyond (16384 x 4096 alone 42.4 / 39.6); 32 x 32 regions 0.8 to 0.95 at any
//     size within the last-level cache;
//   * beyond that cache: 1.12 (16384 x 14336 154 / 173), also where one of the two tensors is (16384 x 1024 x 14336 274 / 281, 32 x 32 regions 264 /
//     284), but not rotated 32 x 32 regions in such a launch (333 / 292).
// Stochastic: both axes 2080 x 1440 18.5 / 11.7, 16384 x 4096 118 / 117, column-wise 16384 x 14336 192 / 182.
struct ColsLaunch {
    bool stochastic, rotated, regions;  // regions: one scale for 32 x 32 elements
    bool both_axes;                     // row-wise outputs too
    int64_t tiles;                      // workgroups of eight waves
    bool some_beyond, all_beyond;       // tensors beyond the last-level cache
};
constexpr int cols_waves(const ColsLaunch &l)
{
    if (l.stochastic) return 4;
    if (l.all_beyond) return 8;
    if (l.regions && l.rotated) return 4;
    if (!l.both_axes) return l.tiles < 512 ? 4 : 8;
    return l.some_beyond || (!l.rotated && l.tiles >= 1536) ? 8 : 4;
}

// dY [M][N] and X [M][K], both column-wise, in one launch: one grid, and one store policy.  (Many tokens of few columns are
// many workgroups: 2^30 tokens of 8 + 8 columns are 2^23, one too many.)
constexpr bool wgrad_operands_share_launch(int64_t M, int64_t N, int64_t K)
{
    const int64_t lim = int64_t(1) << 31;  // (keeps the products below in range)
    return M < lim && N < lim && K < lim && beyond_llc(M, N) == beyond_llc(M, K) &&
           grid_fits(cols_groups(M, N) + cols_groups(M, K), COLS_THREADS);
}

// dY [M][N] both ways and W [N][K] and X [M][K] column-wise in one launch: where both launches would be workgroups of four waves, no
// tensor lies beyond the last-level cache, and one grid holds them.  (Times of both ways stand at the kernel, quantize_backward_kernel.)
constexpr bool backward_operands_share_launch(int64_t M, int64_t N, int64_t K, bool stochastic, bool rotated)
{
    const int64_t lim = int64_t(1) << 31;  // (keeps the products below in range)
    return M < lim && N < lim && K < lim && !beyond_llc(M, N) && !beyond_llc(N, K) && !beyond_llc(M, K) &&
           cols_waves(ColsLaunch{stochastic, rotated, false, true, cols_groups(M, N), false, false}) == 4 &&
           cols_waves(ColsLaunch{stochastic, rotated, false, false, cols_groups(N, K) + cols_groups(M, K), false, false}) == 4 &&
           grid_fits(cols_groups(M, N) + cols_groups(N, K) + cols_groups(M, K), COLS_THREADS);
}

// The smallest forward calls, X [M][K] and W [N][K], in one launch of 32 x 32 tiles.  Up to 256 tiles (one per compute unit) of rows of at most 512
// elements, what the kernel's LDS and registers are laid out for: there it still gains (256 x 512 x 512 in a graph 5.6 / 3.9 us, H32 5.8 / 4.8;
// called from Python 512 x 512 x 512 9.9 / 6.4, 1 x 8192 x 512 9.6 / 6.3), longer rows were not measured.
// Stochastic rounding takes three times as long (512 x 512 x 384 in a graph 7.1 us in two launches, 7.8 in one; 256 x 512 x 512 6.9
// and 9.7) and stops at 256.
constexpr int SMALL_LINEAR_TILE = 32, SMALL_LINEAR_BLOCKS = 16;  // (blocks of 32 elements per row)
constexpr bool small_linear(int64_t M, int64_t N, int64_t K, bool stochastic)
{
    if (M > (1 << 20) || N > (1 << 20) || K > 32 * (stochastic ? SMALL_LINEAR_BLOCKS / 2 : SMALL_LINEAR_BLOCKS)) return false;
    return ((M + SMALL_LINEAR_TILE - 1) / SMALL_LINEAR_TILE) * ((N + SMALL_LINEAR_TILE - 1) / SMALL_LINEAR_TILE) <= 256;
}

}  // namespace mxfp4
