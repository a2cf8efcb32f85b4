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

// dY [M][N] and X [M][K], both column-wise, in one launch: one grid, and one store policy.  (Many tokens of few columns are
// many workgroups: 2^30 tokens of 8 + 8 columns are 2^23, one too many.)
constexpr bool wgrad_operands_share_launch(int64_t M, int64_t N, int64_t K)
{
    const int64_t lim = int64_t(1) << 31;  // (keeps the products below in range)
    return M < lim && N < lim && K < lim && beyond_llc(M, N) == beyond_llc(M, K) &&
           grid_fits(cols_groups(M, N) + cols_groups(M, K), COLS_THREADS);
}

}  // namespace mxfp4
