// The smallest forward calls in one launch: Y = Q(X) Q(W)^T with X and W quantised by the workgroups that multiply them.
//
// What bounds such a call is its launches: at 256 x 512 x 512 the quantiser runs 2.6 us, the product 3.8, and a call took 9.7 us, most of it the
// two launches and the wait of the second for the first.  Here a workgroup owns a 32 x 32 tile of Y: it quantises the tile's 32 rows of X and
// 32 rows of W into LDS (one lane per block, the arithmetic of the row-wise quantiser), multiplies them from there, and the workgroups of
// the first tile column (row) also write X's (W's) codes and scales to the workspace, where a call leaves them.  Every row is
// quantised once per tile beside it, which is why the rule (small_linear) stops at a few blocks per lane.
// us, two launches / one, called from Python and in a graph: 256 x 512 x 512 unrotated 9.8 / 5.9 and 5.6 / 3.9, H32 9.8 / 6.0 and 5.8 / 4.8;
// 256 x 1024 x 128 9.9 / 5.9 and 5.9 / 2.8; 16 x 2048 x 256 stochastic 9.9 / 5.9 and 7.0 / 5.7.
#include "launch_limits.h"
#include "mxfp4_internal.h"
#include "quantize_block.h"

namespace mxfp4 {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int TILE = SMALL_LINEAR_TILE;
constexpr int THREADS = 512;                   // (256: H32, 256 x 512 x 512 5.8 us in a graph, 4.8 with 512)
constexpr int MAX_BLOCKS = SMALL_LINEAR_BLOCKS;
constexpr int PITCH = MAX_BLOCKS * 16 + 16;    // bytes of codes per row in LDS, 16 more than whole banks: 16 rows of one chunk cover them all

struct SmallLinear {
    const uint16_t *x, *w;
    uint8_t *xq, *xs, *wq, *ws;
    void *y;
    int M, N, nkb;  // nkb: blocks per row, K / 32
    uint32_t tiles_n, sign_mask;
    RngKey key_x, key_w;
};

// U: blocks per lane, 64 rows of nkb <= 8 U blocks on 512 lanes
template <int HAD, int RND, bool OUT_FP32, int U>
__global__ __launch_bounds__(THREADS) void linear_small_kernel(const SmallLinear p)
{
    __shared__ __attribute__((aligned(16))) uint8_t codes[2 * TILE * PITCH];
    __shared__ uint8_t scales[2 * TILE][MAX_BLOCKS];
    const int tid = threadIdx.x, nkb = p.nkb;
    const uint32_t tm = blockIdx.x / p.tiles_n, tn = blockIdx.x - tm * p.tiles_n;
    const int m0 = (int)tm * TILE, n0 = (int)tn * TILE;

    // ---- quantise rows 0 .. 31 of X's and 32 .. 63 of W's; rows beyond the matrix are its last one ------------------
    const uint32_t inverse = 65536u / (uint32_t)nkb + 1u;  // (i inverse >> 16 = i / nkb for i < 1024, nkb <= 16)
    uint4 raw[U][4];
    int row_of[U], block_of[U];
    int64_t at[U];  // block of the tensor, -1: none
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t i = (uint32_t)(u * THREADS + tid), r = (i * inverse) >> 16;
        row_of[u] = (int)r;
        block_of[u] = (int)(i - r * (uint32_t)nkb);
        at[u] = -1;
        if (r < 2 * TILE) {
            const bool is_w = r >= TILE;
            const int g = is_w ? n0 + (int)r - TILE : m0 + (int)r, last = (is_w ? p.N : p.M) - 1;
            at[u] = (int64_t)(g < last ? g : last) * nkb + block_of[u];
            const uint4 *src = reinterpret_cast<const uint4 *>(is_w ? p.w : p.x) + at[u] * 4;
#pragma unroll
            for (int j = 0; j < 4; ++j) raw[u][j] = src[j];
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (at[u] < 0) continue;
        const int r = row_of[u], kb = block_of[u];
        const bool is_w = r >= TILE;
        float v[32];
        widen(raw[u], v);
        rotate_block<HAD>(v, p.sign_mask);
        uint4 q;
        uint32_t s;
        encode_scaled<RND>(v, amax_bits(v), is_w ? p.key_w : p.key_x, (uint64_t)at[u] * 32u, q, s);
        *reinterpret_cast<uint4 *>(codes + r * PITCH + kb * 16) = q;
        scales[r][kb] = (uint8_t)s;
        if (is_w ? (tm == 0 && n0 + r - TILE < p.N) : (tn == 0 && m0 + r < p.M)) {
            reinterpret_cast<uint4 *>(is_w ? p.wq : p.xq)[at[u]] = q;
            (is_w ? p.ws : p.xs)[at[u]] = (uint8_t)s;
        }
    }
    // the last instruction's blocks beyond the row's end: zeros under scale 0
    const int padded = (nkb + 3) & ~3;
    if (tid < 2 * TILE)
        for (int kb = nkb; kb < padded; ++kb) {
            *reinterpret_cast<uint4 *>(codes + tid * PITCH + kb * 16) = make_uint4(0, 0, 0, 0);
            scales[tid][kb] = 0;
        }
    __syncthreads();

    // ---- four of the waves, 16 x 16 sums each, contraction ascending --------------------------------------------------------
    if (tid >= 256) return;
    const int lane = tid & 63, wave = tid >> 6, l16 = lane & 15, g = lane >> 4;
    const int ar = 16 * (wave >> 1) + l16, br = TILE + 16 * (wave & 1) + l16;
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < padded; k += 4) {
        const v4i a = *reinterpret_cast<const v4i *>(codes + ar * PITCH + (k + g) * 16);
        const v4i b = *reinterpret_cast<const v4i *>(codes + br * PITCH + (k + g) * 16);
        const v8i a8 = {a.x, a.y, a.z, a.w, 0, 0, 0, 0}, b8 = {b.x, b.y, b.z, b.w, 0, 0, 0, 0};
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b8, a8, acc, 4, 4, 0, (int)scales[br][k + g], 0, (int)scales[ar][k + g]);
    }

    // lane: row l16 of the wave's 16, columns 4 g .. 4 g + 3
    const int row = m0 + ar, col = n0 + 16 * (wave & 1) + 4 * g;
    if (row >= p.M || col >= p.N) return;
    const int64_t to = (int64_t)row * p.N + col;
    const int left = p.N - col;
    if constexpr (OUT_FP32) {
        float *o = static_cast<float *>(p.y) + to;
        if ((p.N & 3) == 0) {
            *reinterpret_cast<v4f *>(o) = acc;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < left) o[e] = acc[e];
        }
    } else {
        uint16_t *o = static_cast<uint16_t *>(p.y) + to;
        const uint32_t lo = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){acc[0], acc[1]}, bf16x2));
        const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){acc[2], acc[3]}, bf16x2));
        if ((p.N & 3) == 0) {
            *reinterpret_cast<uint2 *>(o) = make_uint2(lo, hi);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < left) o[e] = (uint16_t)((e < 2 ? lo : hi) >> (16 * (e & 1)));
        }
    }
}

template <int HAD, int RND, bool OUT_FP32>
void launch_u(const SmallLinear &p, uint32_t tiles, hipStream_t st)
{
    if (p.nkb <= 8) linear_small_kernel<HAD, RND, OUT_FP32, 1><<<tiles, THREADS, 0, st>>>(p);
    else linear_small_kernel<HAD, RND, OUT_FP32, 2><<<tiles, THREADS, 0, st>>>(p);
}

template <int HAD>
void launch_h(const SmallLinear &p, int rounding, int out_fp32, uint32_t tiles, hipStream_t st)
{
    if (rounding == RND_SR) out_fp32 ? launch_u<HAD, RND_SR, true>(p, tiles, st) : launch_u<HAD, RND_SR, false>(p, tiles, st);
    else out_fp32 ? launch_u<HAD, RND_RNE, true>(p, tiles, st) : launch_u<HAD, RND_RNE, false>(p, tiles, st);
}

}  // namespace

hipError_t launch_linear_small(const QuantArgs &x, const QuantArgs &w, void *y, int out_fp32, hipStream_t st)
{
    const uint32_t tiles_n = (uint32_t)((w.rows + TILE - 1) / TILE), tiles = tiles_n * (uint32_t)((x.rows + TILE - 1) / TILE);
    const SmallLinear p{x.x, w.x, x.q, x.s, w.q, w.s, y, (int)x.rows, (int)w.rows, (int)(x.cols / 32), tiles_n, sign_mask_of(x.seed),
                        make_key(x.seed), make_key(w.seed)};
    switch (x.hadamard) {
        case HAD_NONE: launch_h<HAD_NONE>(p, x.rounding, out_fp32, tiles, st); break;
        case HAD_DET: launch_h<HAD_DET>(p, x.rounding, out_fp32, tiles, st); break;
        case HAD_RANDSIGN: launch_h<HAD_RANDSIGN>(p, x.rounding, out_fp32, tiles, st); break;
        case HAD_RANDSIGN16: launch_h<HAD_RANDSIGN16>(p, x.rounding, out_fp32, tiles, st); break;
        default: launch_h<HAD_DET16>(p, x.rounding, out_fp32, tiles, st); break;
    }
    return hipGetLastError();
}

}  // namespace mxfp4
