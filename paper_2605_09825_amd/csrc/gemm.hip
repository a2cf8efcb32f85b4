// Block-scaled FP4 GEMM for gfx950: out[i][j] (+)= sum_c A[i][c] * B[j][c] on MXFP4
// operands (the MXFP4 GEMM of the linear layers, Sec. 1 / App. A.2; operand axes per
// App. C.1-C.3), on the scaled matrix instructions V_MFMA_SCALE_F32_{16X16X128,32X32X64}_F8F6F4.
//
// Register layout of those instructions with FP4 operands (64 lanes, lane = l; n = 16 or 32 rows):
//   first operand : lane l holds row l%n, the 32 K-elements 32*(l/n) .. +31 as 16 bytes
//                   (4 VGPRs), element k in nibble k%32 (low nibble first); its scale VGPR holds
//                   the E8M0 byte of exactly that 32-element block
//   second operand: the same with "row" = output column
//   result        : 16x16: lane l holds column l%16, rows 4*(l/16) + {0..3};
//                   32x32: register e of lane l holds D[8*(e/4) + 4*(l/32) + e%4][l%32]
// i.e. one lane's operand is precisely one MX block of the canonical layout, so the
// canonical q/s arrays feed the instruction without any repacking.
//
// The kernels pass B's rows as the first operand and A's rows as the second: a lane
// then owns 4 consecutive output columns of one output row.
#include <type_traits>

#include "edge_rules.h"
#include "mxfp4_internal.h"
#include "scale_batches.h"

namespace mxfp4 {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    // round to nearest even on the upper 16 bits; NaN keeps a quiet NaN (branch-free)
    const uint32_t u = __float_as_uint(f);
    const uint32_t rounded = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    const uint32_t nan = (u >> 16) | 0x40u;
    return (uint16_t)(((u & 0x7FFFFFFFu) > 0x7F800000u) ? nan : rounded);
}

// two floats -> two bf16 in one dword (first in the low half), round to nearest even: one
// V_CVT_PK_BF16_F32
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// ---- any-shape kernel: operands of different formats, sizes beyond the ragged-shape kernel's grid and offsets, and the
// short products that it is the faster for (see short_product) ----
// 256 threads = 2x2 waves, each wave a 32x32 output tile (2x2 instruction tiles); operands
// come straight from global memory.  Rows beyond the matrix are clamped (their results
// are dropped), K blocks beyond C/32 are fed as zeros.
// AF, BF: element format of each operand, 0 = E2M1 (16 bytes per 32-element block), 1 = E4M3 (32 bytes);
// the instruction's format selectors are 4 for E2M1 and 0 for E4M3.
// One lane's operand registers for the 128 K-elements starting at block k (a multiple of 4), lane group kb.
// E2M1: the lane holds block k + kb, 32 consecutive elements in 16 bytes.  E4M3 (probed on the hardware): the
// lane holds elements 16*kb .. +15 and 64 + 16*kb .. +15 of the 128, 16 bytes each, while its scale register
// still belongs to block k + kb.  Blocks at or beyond nkb read as zeros.
template <int F>
__device__ __forceinline__ v8i load_operand(const uint8_t *q, int64_t row, int64_t C, int64_t nkb, int64_t k, int kb)
{
    const v4i zero = {0, 0, 0, 0};
    if (F == 0) {
        const v4i t = (k + kb < nkb) ? *reinterpret_cast<const v4i *>(q + row * (C >> 1) + (k + kb) * 16) : zero;
        return (v8i){t.x, t.y, t.z, t.w, 0, 0, 0, 0};
    }
    const uint8_t *p = q + row * C + k * 32;
    const v4i t0 = (k + (kb >> 1) < nkb) ? *reinterpret_cast<const v4i *>(p + 16 * kb) : zero;
    const v4i t1 = (k + 2 + (kb >> 1) < nkb) ? *reinterpret_cast<const v4i *>(p + 64 + 16 * kb) : zero;
    return (v8i){t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
}

template <bool OUT_FP32, bool ACC, int AF, int BF>
__global__ __launch_bounds__(256) void gemm_any_kernel(const uint8_t *__restrict__ aq, const uint8_t *__restrict__ as,
                                                       const uint8_t *__restrict__ bq, const uint8_t *__restrict__ bs,
                                                       int64_t Ra, int64_t Rb, int64_t C, void *__restrict__ out,
                                                       int64_t ld)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, kb = lane >> 4;
    const int64_t row0 = (int64_t)blockIdx.x * 64 + (wave >> 1) * 32;
    const int64_t col0 = (int64_t)blockIdx.y * 64 + (wave & 1) * 32;
    const int64_t nkb = C >> 5;

    int64_t ar[2], br[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        int64_t r = row0 + 16 * t + l16, c = col0 + 16 * t + l16;
        ar[t] = r < Ra ? r : Ra - 1;
        br[t] = c < Rb ? c : Rb - 1;
    }
    v4f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

    for (int64_t k = 0; k < nkb; k += 4) {
        const bool kv = k + kb < nkb;
        v8i a[2], b[2];
        int sa[2], sb[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            a[t] = load_operand<AF>(aq, ar[t], C, nkb, k, kb);
            b[t] = load_operand<BF>(bq, br[t], C, nkb, k, kb);
            sa[t] = kv ? as[ar[t] * nkb + k + kb] : 127;
            sb[t] = kv ? bs[br[t] * nkb + k + kb] : 127;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[j], a[i], acc[i][j], BF ? 0 : 4,
                                                                             AF ? 0 : 4, 0, sb[j], 0, sa[i]);
    }

#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t r = row0 + 16 * i + l16;
        if (r >= Ra) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t c = col0 + 16 * j + 4 * kb + e;
                if (c >= Rb) continue;
                float v = acc[i][j][e];
                if (OUT_FP32) {
                    float *o = reinterpret_cast<float *>(out) + r * ld + c;
                    *o = ACC ? (*o + v) : v;
                } else {
                    reinterpret_cast<uint16_t *>(out)[r * ld + c] = f32_to_bf16(v);
                }
            }
        }
    }
}


// ---- tiled kernel: 256 x 256 output tile per workgroup, K consumed in stages of 256 ---------
// 4 waves (2 x 2), each a 128 x 128 sub-tile = 8 x 8 tiles of V_MFMA_SCALE_F32_16X16X128_F8F6F4
// (256 accumulator registers per lane); a narrow variant works on 256 x 128 tiles (sub-tile 128 x 64, 8 x 4
// instruction tiles) with the same data path, see gemm_tile_body.  With FP4 operands that instruction takes, per lane l,
// the 32 K-elements 32*(l/16).. of row l%16 of each operand (one MX block, 16 bytes) and the
// block's scale byte; the result holds, in register e of lane l, D[4*(l/16) + e][l%16].
// The chip is power-limited here (see gemm_tile_body), and this form takes less energy than V_MFMA_SCALE_F32_32X32X64: per
// product it moves half the sums.  Matrix instructions alone, fragments of normal operands in registers: 6.7 PFLOP/s in the 32 x 32 form,
// 7.5 in this one; with a stage's fragment reads from LDS 6.1 and 6.95 (9.9 and 9.85 with all-zero codes, where power plays no part).
// The sums are the same bits.
//
// Data path: packed codes go global -> LDS with the direct-to-LDS loads (no registers), one
// instruction per 8 rows x 128 bytes (whole cache lines: the memory pipeline's cost is per
// request, about 0.45 lines per clock and CU, so partial lines are ruinous).  A wave's 64 lanes
// land at consecutive 16-byte LDS slots, so the lane -> (row, 16-byte chunk) choice on the
// global side fixes the LDS layout; chunk c of row r of an 8-row group g sits at slot
// r*8 + (c ^ r ^ (g&1)), which makes every 16-lane quarter of the later 16-byte fragment reads
// hit all 64 banks once.
// Scale bytes: one row has 8 per stage, far too little for a request of its own, so they
// come in batches of 4 stages (32 bytes per row, two lanes per row), double-buffered; the
// four load instructions of the next batch are spread over the four stages of the current one.
// Two LDS stage buffers; fragments are double-buffered in registers across the 2 K-steps.
// Epilogue: every wave transposes its sub-tile through its own LDS slice so that global
// stores are whole 256- or 512-byte row segments.
constexpr int TILE = 256;                       // output tile edge
constexpr int STAGE_K = 256;                    // K elements per stage = 128 bytes per row
constexpr int OP_BYTES = TILE * STAGE_K / 2;    // 32 KiB per operand and stage
constexpr int STAGE_BYTES = 2 * OP_BYTES;       // 64 KiB
constexpr int OFF_A = 0, OFF_B = OP_BYTES;
constexpr int SCALE_BATCH = 4;                  // stages per scale batch
constexpr int SC_OP_BYTES = TILE * 8 * SCALE_BATCH;  // 8 KiB per operand and batch
constexpr int SC_BUF_BYTES = 2 * SC_OP_BYTES;        // 16 KiB
constexpr int SC_PIECE_BYTES = SC_OP_BYTES / 2;      // half an operand's rows: 4 KiB
constexpr int OFF_SC = 2 * STAGE_BYTES;              // scale buffers behind the two stage buffers
constexpr int LDS_BYTES = 2 * STAGE_BYTES + 2 * SC_BUF_BYTES;  // 163840 = all of the CU's LDS
constexpr int GROUP_M = 4;                      // tile rows per rasterisation group
constexpr int NUM_CUS = 256;                    // MI355X: 8 XCDs x 32 CUs

typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ void dma16(uint32_t lds_addr, uint32_t voff, const uint8_t *sbase)
{
    // each lane: 16 bytes from sbase + voff to LDS[lds_addr + 16*lane] (the ISA wants one wait state between a
    // scalar write of M0 and a direct-to-LDS load that reads it)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\t" ::"s"(lds_addr), "v"(voff), "s"(sbase)
                 : "memory");
}

// A run of such loads under one M0: each lane's 16 bytes from sbase + voff + IMM to LDS[M0 + IMM + 16*lane] (the
// instruction's immediate offset moves both addresses; -4096 <= IMM < 4096).  Only the first load of a run
// (SETM0) writes M0 = lds_base.
template <int IMM, bool SETM0>
__device__ __forceinline__ void dma16_run(uint32_t lds_base, uint32_t voff, const uint8_t *sbase)
{
    static_assert(IMM >= -4096 && IMM < 4096, "13-bit signed instruction offset");
    if (SETM0)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3\n\t" ::"s"(lds_base),
                     "v"(voff), "s"(sbase), "n"(IMM)
                     : "memory");
    else
        asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2\n\t" ::"v"(voff), "s"(sbase), "n"(IMM) : "memory");
}

template <int V>
using IC = std::integral_constant<int, V>;

// Operand rows one wave loads for one tile: rows wave*64 .. +63 of the tile's A rows, B rows and
// of their scale rows.
struct TileSrc {
    const uint8_t *a, *b, *as, *bs;
    int64_t m0, n0;
    int dm, dn;  // RAG: rows and columns at the tile's start that belong to its neighbours
};

// Slots behind a stage's barrier (see gemm_tile_body): the step of settling the next stage's scales that goes in front of the slot-th matrix
// instruction from there, -1: none.  One a slot; wide tile: two in every four slots, then three.
template <int FMT, int NJ>
constexpr int settle_step(int slot)
{
    if (FMT) return slot >= 17 && slot < 25 ? slot - 17 : -1;
    if (NJ == 2) return slot >= 11 && slot < 23 ? slot - 11 : -1;
    if (slot < 33) return slot < 19 ? -1 : slot % 4 == 3 ? (slot - 19) / 2 : slot % 4 == 0 ? (slot - 20) / 2 + 1 : -1;
    return slot >= 34 && slot < 44 && slot % 4 != 1 ? 8 + (slot - 34) / 4 * 3 + (slot - 34) % 4 : -1;
}
// every step once, in order, and two matrix instructions between the last and the first one of the next stage, which reads what it leaves
template <int FMT, int NJ>
constexpr bool settled_in_time(int slots, int steps)
{
    int next = 0, last = slots;
    for (int slot = 0; slot < slots; ++slot) {
        if (settle_step<FMT, NJ>(slot) < 0) continue;
        if (settle_step<FMT, NJ>(slot) != next) return false;
        ++next;
        last = slot;
    }
    return next == steps && last + 2 <= slots;
}

// 16 or 8 bytes at any address
struct __attribute__((packed, aligned(1))) Bytes16 { uint32_t v[4]; };
struct __attribute__((packed, aligned(1))) Bytes8 { uint32_t v[2]; };
struct __attribute__((packed, aligned(1))) Bytes4 { uint32_t v; };

// The whole tiled GEMM as seen by one workgroup: `wg` of `nwg` workgroups share the problem (the ids are
// virtual: a launch may run two problems side by side on disjoint sets of CUs).  smem: the workgroup's
// LDS_BYTES of LDS, lds0 its LDS address.
// FMT: element format of both operands.  0 = E2M1: a stage (128 bytes per row) holds 256 K-elements = 2
// instruction K-steps, one fragment (16 bytes per lane) each.  1 = E4M3: a stage holds 128 K-elements = 1
// instruction K-step of 32 bytes per lane.  The instruction wants, from lane group g, the elements 16g .. +15
// and 64 + 16g .. +15 of its 128 (probed), which are exactly the two 16-byte fragments the E2M1 path fetches
// for its K-steps 0 and 1: so data movement, LDS layout and fragment reads are the same for both formats,
// and only the matrix instructions differ (half as many, taking two fragments each).
// NJ: 32-column groups of a wave's sub-tile.  4: the 256 x 256 tile (wave sub-tile 128 x 128, 64 matrix
// instructions per K-step).  2 (E2M1 only): a 256 x 128 tile (sub-tile 128 x 64, 32 instructions per K-step) for
// outputs that have too few 256 x 256 tiles to fill the chip, and for the part-filled last round of others;
// it moves 1.5 times the operand bytes per flop, so it is only used where compute units would idle otherwise.
// l_lo, l_hi: the body works on tiles l_lo .. l_hi-1 of the tile sequence only (l_hi < 0: all of them).
// HALVES (narrow tile only): tiles_n and the sequence are those of the 256 x 256 grid, and every one of those
// tiles is worked on as two 256 x 128 tiles, left half then right half: the part-filled last round of a launch
// that ran its whole rounds on 256 x 256 tiles.
// RAG: Ra >= 256 rows and Rb >= 256 columns in no whole tiles, C >= 1024 in no whole stages.  The last tile row and
// column are moved back to end with the matrix and store only what is theirs; the last stage is moved back to end with
// the row, and the scale bytes of the blocks it repeats are set to 0 in both operands (products below 2^-254 * 2^24: 0
// in fp32).  Scale rows then start at any byte, so they go through registers: a 16-byte load per lane takes the place of
// every direct-to-LDS scale load, and its bytes are written to LDS one stage later, right behind the barrier that has
// waited for all loads anyway; hence the loads run two stages ahead, not one.
// What bounds it: power.  With normal operands the clock settles at 1.7 to 1.8 GHz (2.4 with all-zero codes), and whatever moves data costs
// clock: without the operand loads 8192 x 6144 x 16384 takes 276 us instead of 322, without the fragment reads no less.  Beside that every
// instruction between two matrix instructions counts (16 clocks each, three others fit): taking the scalar arithmetic of a stage from 70 to
// 25 instructions, in idle slots, gave 322 -> 311 us.  us, in the 32 x 32 form / this one, both on one card: bf16 8192 x 6144 x 4096 93.8 /
// 89.3, x 16384 313.7 / 298.4 (5.53 PFLOP/s); fp32 6144 x 4096 x 8192 95.7 / 92.9, 4096 x 4096 x 8192 added to 71.5 / 68.7; narrow tiles
// 8192 x 1024 x 4096 20.2 / 19.7; MXFP8 8192 x 8192 x 4096 202 / 187 (2.94 PFLOP/s).  The power control's state counts: on another card,
// 2.5 s back to back and, in brackets, the 20 launches soon after a second's pause: 8192 x 6144 x 4096 99.3 / 95.6 (103.5 / 98.0),
// x 16384 339.5 / 320.5 (392.8 / 386.6); MXFP8 8192 x 6144 x 4096 161.1 / 149.2 (190.5 / 174.9).
template <bool OUT_FP32, bool ACC, int FMT, int NJ, bool HALVES = false, bool RAG = false>
__device__ __forceinline__ void gemm_tile_body(const uint8_t *__restrict__ aq, const uint8_t *__restrict__ as,
                                               const uint8_t *__restrict__ bq, const uint8_t *__restrict__ bs,
                                               int64_t C, void *__restrict__ out, int64_t ld, int tiles_m,
                                               int tiles_n, const uint32_t wg, const uint32_t nwg,
                                               uint8_t *const smem, const uint32_t lds0, const int l_lo = 0,
                                               const int l_hi = -1, const int64_t Ra = 0, const int64_t Rb = 0)
{
    static_assert(!HALVES || NJ == 2, "only the narrow tile works on halves of 256 x 256 tiles");

    static_assert(NJ == 4 || (NJ == 2 && FMT == 0), "the narrow tile is built for E2M1 operands only");
    constexpr int TILE_N = 64 * NJ;          // B rows (output columns) per tile
    constexpr int BROWS = TILE_N / 4;        // B rows one wave loads per stage: 64 or 32
    constexpr int NLOADS = 8 + BROWS / 8;    // direct-to-LDS loads per wave and stage: 16 or 12
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t rowbytes = FMT ? C : (C >> 1), nkb = C >> 5;
    const int nstages = (int)((rowbytes + (RAG ? STAGE_K / 2 - 1 : 0)) / (STAGE_K / 2));  // >= 4 (E2M1) or >= 8 (E4M3): the host checks
    constexpr int BATCH = FMT ? 8 : 4;   // stages per scale batch (32 scale bytes per row)
    constexpr int SC_STAGE = FMT ? 4 : 8;  // scale bytes per row and stage

    // ---- persistent tile schedule -----------------------------------------------------------
    // Workgroup ids are dealt round-robin to the 8 XCDs (each with its own L2).  XCD x owns a
    // contiguous run of the tile sequence; its workgroups walk that run with a stride equal to
    // their number, so the tiles in flight on one XCD are consecutive in the sequence, and the
    // sequence goes through the tile grid in groups of GROUP_M tile rows: those tiles share
    // A and B panels in the XCD's L2.
    const int T = ((l_hi < 0 ? tiles_m * tiles_n : l_hi) - l_lo) * (HALVES ? 2 : 1), G = (int)nwg;
    const int xcd = wg & 7, lw = wg >> 3;
    const int nwg_x = (G - xcd + 7) >> 3;                      // workgroups living on this XCD
    const int per = T >> 3, rem = T & 7;
    const int count_x = per + (xcd < rem ? 1 : 0);             // tiles owned by this XCD
    const int start_x = xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per;
    auto tile_src = [&](int lloc) {
        const int Lr = start_x + lloc;                       // position in this body's range
        const int L = l_lo + (HALVES ? (Lr >> 1) : Lr);      // position in the tile sequence
        const int span = GROUP_M * tiles_n, grp = L / span, first = grp * GROUP_M;
        const int gm = (tiles_m - first) < GROUP_M ? (tiles_m - first) : GROUP_M;
        const int in = L - grp * span;
        TileSrc t;
        t.m0 = (int64_t)(first + in % gm) * TILE;
        t.n0 = HALVES ? (int64_t)(in / gm) * TILE + (Lr & 1) * TILE_N : (int64_t)(in / gm) * TILE_N;
        t.dm = t.dn = 0;
        if (RAG) {
            const int64_t mx = Ra - TILE, nx = Rb - TILE_N;
            if (t.m0 > mx) t.dm = (int)(t.m0 - mx), t.m0 = mx;
            if (t.n0 > nx) t.dn = (int)(t.n0 - nx), t.n0 = nx;
        }
        t.a = aq + (t.m0 + wave * 64) * rowbytes;
        t.b = bq + (t.n0 + wave * BROWS) * rowbytes;
        t.as = as + (t.m0 + wave * 64) * nkb;
        t.bs = bs + (t.n0 + wave * BROWS) * nkb;
        return t;
    };
    if (lw >= count_x) return;  // (whole workgroup: nothing to do)

    // ---- direct-to-LDS loads: per-lane offsets (fixed for the whole kernel) -----------------
    // dvo[g]: this lane's 16 bytes of 8-row group g of the wave's 64 rows (row 8g + lane/8; the chunk within
    // the row's 128 bytes is swizzled by the row, odd groups one further)
    const int drr = lane >> 3, dcc = lane & 7;
    uint32_t dvo[8];
#pragma unroll
    for (int g = 0; g < 8; ++g)  // (less the immediate offset (g - 4) KiB the load instruction adds back)
        dvo[g] = (uint32_t)((8 * g + drr) * rowbytes) + (uint32_t)((dcc ^ drr ^ (g & 1)) << 4) - (uint32_t)((g - 4) * 1024);
    // the wave's 8 x 1 KiB of A's stage slice and 8 (narrow tile: 4) x 1 KiB of B's
    const uint32_t lds_wave_a = lds0 + OFF_A + (uint32_t)wave * 8192u;
    const uint32_t lds_wave_b = lds0 + OFF_B + (uint32_t)wave * (uint32_t)(BROWS * 128);
    const uint32_t svoff = (uint32_t)((lane >> 1) * nkb) + (uint32_t)((lane & 1) << 4);

    // load n (0..15) of a stage for this wave, in issue order: n = 0..3 A's 8-row groups 0..3,
    // 4..7 B's groups 0..3, 8..11 A's groups 4..7, 12..15 B's groups 4..7 (the narrow tile has no 12..15: a
    // wave loads only 32 rows of B).  The four loads of a run share one M0
    // (the LDS address of the operand's group 4; the groups sit at immediate offsets (g - 4) KiB from it);
    // `force` makes a load set M0 itself (where scale loads, which set their own, are issued in between).
    // ld_a, ld_b, ld_buf: the stage being loaded and the offset of the stage buffer it goes to; both move on once per stage, in phase 1.
    const uint8_t *ld_a = nullptr, *ld_b = nullptr;
    uint32_t ld_buf = 0;
    int64_t ld_k = 0;  // RAG: the stage's offset in a row
    auto issue_load = [&](auto nc, auto force) {
        constexpr int n = decltype(nc)::value, op = (n >> 2) & 1, g = (n >> 3) * 4 + (n & 3);
        static_assert(n < NLOADS, "no such load for this tile shape");
        constexpr bool setm0 = decltype(force)::value || (n & 3) == 0;
        dma16_run<(g - 4) * 1024, setm0>((op ? lds_wave_b : lds_wave_a) + 4096 + ld_buf, dvo[g], op ? ld_b : ld_a);
    };
    const int64_t k_last = rowbytes - STAGE_K / 2;
    auto set_load = [&](const TileSrc &t, int s) {  // (s = 0 or 1; every row has more stages)
        ld_k = s * (STAGE_K / 2);
        ld_a = t.a + ld_k, ld_b = t.b + ld_k;
    };
    using no_force = std::false_type;
    using force_m0 = std::true_type;
    // Scale batch b holds the 32 scale bytes per row of stages first(b) .. first(b)+3, where
    // first(b) = min(4b, nstages-4): the last batch is pulled back so that it never reads past a
    // row's end (batches past the end of K just repeat the last one into the idle buffer).
    auto batch_first = [&](int b) { return (BATCH * b < nstages - BATCH) ? BATCH * b : nstages - BATCH; };
    // instruction j (0..3) of batch b for this wave: j>>1 = operand, j&1 = which 32 of its 64 rows
    // Batch b of a tile lives in scale buffer (b ^ par) & 1; par alternates between tiles so that
    // a tile's first batch never lands in the buffer its predecessor's last batch is still read from.
    // Its 1 KiB (32 rows x 32 bytes) lie at piece j, wave: so that the place follows from the counter of stages in two operations.
    // (narrow tile: a wave has only 32 rows of B, so instruction 3 repeats instruction 2: the same bytes again, which keeps the stage
    // bodies free of branches)
    auto scales_dst = [&](int b, int j, int par) {
        if (NJ == 2 && j == 3) j = 2;
        return lds0 + OFF_SC + ((b ^ par) & 1) * SC_BUF_BYTES + j * SC_PIECE_BYTES + wave * 1024;
    };
    auto scales_src = [&](const TileSrc &t, int b, int j) {
        if (NJ == 2 && j == 3) j = 2;
        return ((j >> 1) ? t.bs : t.as) + (int64_t)(j & 1) * 32 * nkb + batch_first(b) * SC_STAGE;
    };
    auto issue_scales = [&](const TileSrc &t, int b, int j, int par) {
        dma16(scales_dst(b, j, par), svoff, scales_src(t, b, j));
    };

    // RAG: the same pieces through registers; sp[4] is the piece on its way in the steady state
    uint4 sp[5];
    auto rag_first = [&](int b) { return 32 * b < (int)nkb - 32 ? 32 * b : (int)nkb - 32; };  // first byte of a batch
    auto rag_load = [&](const TileSrc &t, int b, int j) {
        if (NJ == 2 && j == 3) j = 2;
        const uint8_t *src = ((j >> 1) ? t.bs : t.as) + (int64_t)(j & 1) * 32 * nkb + rag_first(b);
        const Bytes16 v = *reinterpret_cast<const Bytes16 *>(src + svoff);
        return make_uint4(v.v[0], v.v[1], v.v[2], v.v[3]);
    };
    auto rag_store = [&](int b, int j, int par, const uint4 &v) {
        *reinterpret_cast<uint4 *>(smem + (scales_dst(b, j, par) - lds0) + lane * 16) = v;
    };

    // ---- fragment reads: per-lane offsets ---------------------------------------------------
    // Lane l of an instruction holds row l % 16 of its 16 and block l / 16 of its four.
    constexpr int NB = 2 * NJ;  // 16-column groups of the wave's sub-tile (its rows: 8 groups)
    const int fr = lane & 15, fg = lane >> 4;
    const int fm = (fr & 7) ^ (fr >> 3);
    const uint32_t fl0 = (uint32_t)((fr >> 3) * 1024 + (fr & 7) * 128);
    // LDS offsets of this lane's piece of A's and B's first fragment in K-step kk, in the buffer of the stage whose fragments are next
    uint32_t ra[2], rb[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        const uint32_t f = fl0 + (uint32_t)((((kk << 2) | fg) ^ fm) << 4);
        ra[kk] = f + OFF_A + wm * 16 * 1024;
        rb[kk] = f + OFF_B + wn * (NJ * 4) * 1024;
    }
    auto other_buffer = [&](uint32_t &at) {
        at ^= STAGE_BYTES;
        asm volatile("" : "+v"(at));
    };
    // RAG: keeps the scale bytes of the blocks that the last stage does not repeat (bytes as settle_scales leaves them)
    uint32_t last_mask = 0xFFFFFFFFu;
    if (RAG) {
        const int again = nstages * SC_STAGE - (int)nkb;
        if (fg < again) last_mask = FMT ? 0u : 0xFFFF0000u;
        if (!FMT && 4 + fg < again) last_mask = 0u;
    }
    // (the wave's 64-row pieces of A, and of B on the wide tile, were loaded by one wave in two halves; the narrow tile's by two waves)
    const uint32_t sa_row0 = OFF_SC + wm * 2048 + (lane >> 5) * SC_PIECE_BYTES + (lane & 31) * 32;
    const uint32_t sb_row0 = OFF_SC + SC_OP_BYTES + wn * 2048 + (lane >> 5) * (NJ == 4 ? SC_PIECE_BYTES : 1024) + (lane & 31) * 32;

    v4i fa[2][8], fb[2][NB];
    // Scale bytes of a stage.  A lane reads those of ONE row, 64 rows (four fragments) per instruction, and the wave then turns the 4 x 4
    // square of (fragment, block) over its four lane groups, so that lane group g holds block g of all four; the instruction's byte
    // selector picks the fragment.  (Read per fragment, by all four lane groups alike, they took a fifth of the LDS' time.)
    // E2M1: set q = 0, 1: A's rows 64 q .. +63; 2, 3: B's.  word (q, f & 1): bytes {K-step 0: fragments f, f + 2; K-step 1: f, f + 2}.
    // E4M3: set 0: A, 1: B.  word (q, f & 1): bytes {fragments f, f + 2, f + 4, f + 6}.
    constexpr int SETS = FMT ? 2 : 2 + NJ / 2;
    uint32_t sc_cur[SETS][2], sc_old[SETS][2];  // (sc_old: for phases 2 and 3, while the next stage's arrive in sc_cur)
    uint32_t raw[SETS][2];
    // One fragment: rows 16 i .. 16 i + 15 of the wave's part of A or B, 16-byte chunks 4 kk .. 4 kk + 3.
    auto read_a = [&](int kk, int i) { fa[kk][i] = *reinterpret_cast<const v4i *>(smem + ra[kk] + i * 2048); };
    auto read_b = [&](int kk, int j) { fb[kk][j] = *reinterpret_cast<const v4i *>(smem + rb[kk] + j * 2048); };
    const int sb_lim = RAG ? (int)nkb - 32 : (nstages - BATCH) * SC_STAGE;  // byte of a row's scales where the last batch begins
    // piece n (0 .. 3; the narrow tile has no 3): A's rows 0 .. 63, B's, A's 64 .. 127, B's
    auto read_scales = [&](uint32_t place, int n) {
        const uint8_t *p = smem + (((n & 1) ? sb_row0 : sa_row0) + place) + (n >> 1) * 1024;
        if (FMT) {
            raw[n & 1][n >> 1] = reinterpret_cast<const Bytes4 *>(p)->v;
        } else {
            const int q = (n & 1) * 2 + (n >> 1);
            if constexpr (RAG) {
                const Bytes8 v = *reinterpret_cast<const Bytes8 *>(p);
                raw[q][0] = v.v[0], raw[q][1] = v.v[1];
            } else {
                const uint2 v = *reinterpret_cast<const uint2 *>(p);
                raw[q][0] = v.x, raw[q][1] = v.y;
            }
        }
    };
    // Step 0 .. 3 of turning set q; `last`: these are the scales of a tile's last stage.  raw = two words x, y of bytes 0 .. 3 of the row.
    auto settle_scales = [&](int q, int step, bool last) {
        uint32_t *r = raw[q];
        if (step == 0) {  // {x0, x1, y0, y1} and {x2, x3, y2, y3}
            const uint32_t x = r[0], y = r[1];
            r[0] = __builtin_amdgcn_perm(y, x, 0x05040100u);
            r[1] = __builtin_amdgcn_perm(y, x, 0x07060302u);
        } else if (step == 1) {  // lane groups 0, 1 and 2, 3: the first word of the upper for the second of the lower
            const auto w = __builtin_amdgcn_permlane32_swap(r[0], r[1], false, false);
            r[0] = w[0], r[1] = w[1];
        } else if (step == 2) {
            const uint32_t x = r[0], y = r[1];
            r[0] = __builtin_amdgcn_perm(y, x, 0x06020400u);
            r[1] = __builtin_amdgcn_perm(y, x, 0x07030501u);
        } else {  // lane groups 0, 2 and 1, 3
            const auto w = __builtin_amdgcn_permlane16_swap(r[0], r[1], false, false);
            sc_cur[q][0] = w[0], sc_cur[q][1] = w[1];
            if (RAG && last) sc_cur[q][0] &= last_mask, sc_cur[q][1] &= last_mask;
        }
    };
    // E2M1: the sets in the order their bytes are read in
    auto settle_set = [](int n) { return (n & 1) * 2 + (n >> 1); };
    // (opaque: as a plain assignment the compiler keeps one register and copies all of them at the end of a stage)
    auto age_scales = [&](int n) { asm volatile("v_mov_b32 %0, %1" : "=v"(sc_old[n >> 1][n & 1]) : "v"(sc_cur[n >> 1][n & 1])); };

    // Stage s of a tile lives in stage buffer (s & 1) ^ bp.  The hand-over loads put the next tile's stage 0
    // into the buffer after the current tile's last one, so with an odd number of stages the parity flips
    // from tile to tile.
    int bp = 0;
    v4f acc[8][NB];

    // One matrix instruction: tile (I, J) of the wave's 8 x NB, fragments and scale bytes of K-step KK.  In assembly, so that the sum stays
    // where it is: with four registers per sum and none to spare the compiler moves a quarter of them about at every change of stage body.
    // What the compiler then leaves to this code, and every change of it has to keep:
    //   * two wait states between a vector instruction and a matrix instruction that reads its result: the scales, which are settled at least
    //     two matrix instructions ahead (settled_in_time) and aged a phase ahead, and any copy that the compiler puts at a change of stage body
    //     (the wait that every stage body begins with; its time does not show: 8192 x 6144 x 4096 forward and backward 345.2 / 345.3 us);
    //   * 19 between a matrix instruction and anything but itself that touches its sums: the wait before the epilogue reads them (below).
    // The fragments come from LDS, for whose loads the compiler waits.  tests/test_codegen.py looks for both in the built library.
#define MXFP4_MFMA(FIRST, SECOND, SB, SA, SELB, SELA, FORMATS, FRESH)                                            \
    if constexpr (FRESH)                                                                                        \
        asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, 0, %3, %4 op_sel:[%5,%6,0] op_sel_hi:[%7,%8,0]" FORMATS \
                     : "=a"(acc[i_][j_])                                                                        \
                     : "v"(FIRST), "v"(SECOND), "v"(SB), "v"(SA), "n"((SELB) & 1), "n"((SELA) & 1), "n"((SELB) >> 1), "n"((SELA) >> 1)); \
    else                                                                                                        \
        asm volatile("v_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel:[%5,%6,0] op_sel_hi:[%7,%8,0]" FORMATS \
                     : "+a"(acc[i_][j_])                                                                        \
                     : "v"(FIRST), "v"(SECOND), "v"(SB), "v"(SA), "n"((SELB) & 1), "n"((SELA) & 1), "n"((SELB) >> 1), "n"((SELA) >> 1));
    // Instruction G of phase P (GAPS of them).  E2M1: phase P is K-step P/2 on rows 64 (P%2) .. +63 of the sub-tile, columns to and fro, so
    // that consecutive instructions share a fragment.  E4M3 (instructions twice as long; both fragments of a row are one K-step's): phase P
    // is the quarter (P/2, P%2) of the sub-tile.
#define MXFP4_SLOT_MMA(P, G, MODE)                                                                              \
    if constexpr (FMT == 0 && (G) < GAPS) {                                                                     \
        constexpr int kk_ = (P) >> 1, i_ = 4 * ((P) & 1) + (G) / NB, c_ = (G) % NB, j_ = (i_ & 1) ? NB - 1 - c_ : c_; \
        constexpr int qb_ = 2 + (j_ >> 2), qa_ = i_ >> 2;                                                       \
        MXFP4_MFMA(fb[kk_][j_], fa[kk_][i_], (kk_ ? sc_old[qb_][j_ & 1] : sc_cur[qb_][j_ & 1]),                  \
                   (kk_ ? sc_old[qa_][i_ & 1] : sc_cur[qa_][i_ & 1]), 2 * kk_ + ((j_ >> 1) & 1), 2 * kk_ + ((i_ >> 1) & 1), \
                   " cbsz:4 blgp:4", (MODE) == 3 && (P) < 2)                                                    \
    }                                                                                                           \
    if constexpr (FMT == 1 && (G) < GAPS) {                                                                     \
        constexpr int i_ = 4 * ((P) >> 1) + ((G) >> 2) % 4, j_ = 4 * ((P) & 1) + ((G) & 3);                      \
        const v8i fb8 = {fb[0][j_].x, fb[0][j_].y, fb[0][j_].z, fb[0][j_].w, fb[1][j_].x, fb[1][j_].y, fb[1][j_].z, fb[1][j_].w}; \
        const v8i fa8 = {fa[0][i_].x, fa[0][i_].y, fa[0][i_].z, fa[0][i_].w, fa[1][i_].x, fa[1][i_].y, fa[1][i_].z, fa[1][i_].w}; \
        MXFP4_MFMA(fb8, fa8, ((P) < 2 ? sc_cur[1][j_ & 1] : sc_old[1][j_ & 1]), ((P) < 2 ? sc_cur[0][i_ & 1] : sc_old[0][i_ & 1]), \
                   (j_ >> 1), (i_ >> 1), "", (MODE) == 3)                                                       \
    }
#define MXFP4_PIN() __builtin_amdgcn_sched_barrier(0);
    constexpr int GAPS = FMT ? 16 : 8 * NJ;  // matrix instructions per phase
    // The barrier stands in front of this instruction of phase 2.  Loads of the stage after next go out from there on, LOADS_LATE of them up to
    // the stage's end and the rest in the next one's phase 0.
    constexpr int BAR = FMT ? 4 : NJ == 4 ? 14 : 8, LATE_GAPS = 2 * GAPS - BAR, LOADS_LATE = NJ == 4 ? 12 : 8;
    static_assert(settled_in_time<FMT, NJ>(LATE_GAPS, 4 * SETS), "scales are read by the matrix instruction behind them too early");
    // item of a list of `count` that goes in front of instruction G, one every `step` from `first` on; -1: none
#define MXFP4_AT(G, FIRST, STEP, COUNT) ((G) >= (FIRST) && ((G) - (FIRST)) % (STEP) == 0 && ((G) - (FIRST)) / (STEP) < (COUNT) ? ((G) - (FIRST)) / (STEP) : -1)
#define MXFP4_32(M) M(0) M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15) \
    M(16) M(17) M(18) M(19) M(20) M(21) M(22) M(23) M(24) M(25) M(26) M(27) M(28) M(29) M(30) M(31)
#define MXFP4_16(M) M(0) M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15)
    // The fragments fetched in each part of a stage, in order (n-th of its list); `late`, behind the barrier, are the next stage's first.
    //   E2M1     late: A0, all of B, A1 (K-step 0) | phase 0: A2 .. A7, (wide tile:) K-step 1's B0, B1 | 1: the rest of B, A0 .. A3 | 2: A4 .. A7
    //   E4M3     late: A0 .. A3, in phase 3 B0 .. B3, two halves each | phase 0: B4 .. B7 | 1: A4 .. A7
    constexpr int LATE = 3;
    auto fetch = [&](int part, int n) {
        if (FMT) {
            const int f = n >> 1, h = n & 1;
            if (part == LATE) { if (f < 4) read_a(h, f); else read_b(h, f - 4); }
            if (part == 0) read_b(h, 4 + f);
            if (part == 1) read_a(h, 4 + f);
        } else {
            constexpr int EARLY = NJ == 4 ? 2 : 0;  // fragments of K-step 1's B that phase 0 fetches
            if (part == LATE) { if (n >= 1 && n <= NB) read_b(0, n - 1); else read_a(0, n ? 1 : 0); }
            if (part == 0) { if (n < 6) read_a(0, 2 + n); else read_b(1, n - 6); }
            if (part == 1) { if (n < NB - EARLY) read_b(1, EARLY + n); else read_a(1, n - (NB - EARLY)); }
            if (part == 2) read_a(1, 4 + n);
        }
    };

    // One stage = 4 phases of 32 matrix instructions (narrow tile: 16; E4M3: 16, twice as long).  Everything else is
    // threaded between them, evenly, and pinned there with scheduling barriers: with a single
    // wave per SIMD any stall of the wave (a burst of loads filling the memory pipeline's queue,
    // a late fragment) idles the matrix unit, and an instruction of 16 clocks covers three others.
    //   phase 0: the rest of the next stage's direct-to-LDS loads
    //   phases 0, 1, 2: fragments (see fetch)
    //   barrier in phase 2 (this stage's buffer is free, the next stage has landed)
    //   behind it: the next stage's first fragments and its scales; most of the loads of
    //              the stage after next, into the buffer just freed; one scale load
    // The main loop's body must stay one basic block (no data-dependent branches), or the matrix
    // instructions get sunk behind the branches; so the last two stages of a tile, which hand
    // over to the next tile, are separate instantiations (MODE 1 and 2).
    //   MODE 3: stage 0: as MODE 0, and every accumulator's first instruction starts from zero
    //   MODE 0: stage 1 <= s <= nstages-3 of tile `cur`
    //   MODE 1: stage nstages-2: behind its barrier it starts loading stage 0 and scale batch 0 of tile `nxt`
    //   MODE 2: stage nstages-1: its phase 0 finishes stage 0; behind the barrier it issues the first load of
    //           nxt's scale batch 1 and fetches nothing (the epilogue follows)
    auto stage = [&](const TileSrc &cur, const TileSrc &nxt, int par, int par_nxt, int s, auto mode) {
        constexpr int MODE = decltype(mode)::value;
        asm volatile("s_nop 1");  // (no vector instruction's result is read before this has passed, see MXFP4_MFMA)
        __builtin_amdgcn_sched_barrier(0);
        // Place of the next stage's scales (behind sa_row0 or sb_row0), and destination and source of this stage's one scale load (piece (s + 1) & 3 of the batch after
        // that of stage s + 1): worked out a step at a time in idle slots of phase 1, used in phase 3.
        uint32_t sc_next = 0, sc_dst = 0, sc_off = 0;
        const uint8_t *sc_src = nullptr;
        const int sb = SC_STAGE * (s + 1);
        constexpr bool STEADY = MODE == 0 || MODE == 3;
        auto step = [&](int n) {
            if (n == 0 && MODE != 2) {
                if (MODE == 1) ld_a = nxt.a;
                else if (RAG) ld_k = ld_k + STAGE_K / 2 < k_last ? ld_k + STAGE_K / 2 : k_last, ld_a = cur.a + ld_k;
                else ld_a += STAGE_K / 2;
                asm volatile("" : "+s"(ld_a));
            }
            if (n == 1 && MODE != 2) {
                if (MODE == 1) ld_b = nxt.b;
                else if (RAG) ld_b = cur.b + ld_k;
                else ld_b += STAGE_K / 2;
                asm volatile("" : "+s"(ld_b));
                ld_buf ^= STAGE_BYTES;
                asm volatile("" : "+s"(ld_buf));
            }
            if (n == 2 && MODE != 2) {
                const int first = (sb & ~31) < sb_lim ? (sb & ~31) : sb_lim;
                sc_next = (uint32_t)((RAG && sb > (int)nkb - SC_STAGE ? (int)nkb - SC_STAGE : sb) - first);
                asm volatile("" : "+s"(sc_next));
            }
            if (n == 3 && MODE != 2) {
                sc_next += (uint32_t)(((sb & 32) << 9) ^ (par << 14));
                asm volatile("" : "+s"(sc_next));
            }
            if (n == 4 && !RAG && STEADY) {
                const int first = (sb & ~31) + 32;
                sc_off = (uint32_t)(first < sb_lim ? first : sb_lim);
                asm volatile("" : "+s"(sc_off));
            }
            if (n == 5 && !RAG && STEADY) {
                sc_dst = FMT ? (uint32_t)(((sb & 12) << 10) | ((sb & 32) << 9)) : (uint32_t)((sb & 56) << 9);
                asm volatile("" : "+s"(sc_dst));
                sc_dst = (sc_dst ^ (uint32_t)(((par ^ 1) << 14))) + lds0 + OFF_SC + wave * 1024;
                asm volatile("" : "+s"(sc_dst));
            }
            if (n == 6 && !RAG && STEADY) {
                sc_src = (sb & 2 * SC_STAGE) ? cur.bs : cur.as;
                asm volatile("" : "+s"(sc_src));
            }
            if (n == 7 && !RAG && STEADY) {  // (narrow tile: piece 3 is piece 2 again)
                const bool second = (sb & SC_STAGE) && !(NJ == 2 && (sb & 2 * SC_STAGE));
                sc_off += second ? (uint32_t)(32 * nkb) : 0u;
                asm volatile("" : "+s"(sc_off));
            }
        };
        // Behind the barrier, in front of the L-th instruction from there (LATE_GAPS of them, of phases 2 and 3)
        auto late = [&](auto l) {
            constexpr int L = decltype(l)::value, P3 = L - (GAPS - BAR);
            constexpr int f_ = FMT ? (P3 < 0 ? MXFP4_AT(L, 2, 1, 8) : P3 < 8 ? 8 + P3 : -1) : NJ == 4 ? MXFP4_AT(L, 5, 4, 10) : MXFP4_AT(L, 4, 3, 6);
            constexpr int r_ = FMT ? MXFP4_AT(L, 1, 2, 4) : NJ == 4 ? MXFP4_AT(L, 4, 4, 4) : MXFP4_AT(L, 1, 2, 3);
            constexpr int d_ = FMT ? MXFP4_AT(L, 1, 2, 12) : NJ == 4 ? MXFP4_AT(L, 2, 4, 12) : MXFP4_AT(L, 0, 3, 8);
            constexpr int w_ = MXFP4_AT(L, 0, 2, 5);  // RAG: scale piece on its way
            constexpr int t_ = settle_step<FMT, NJ>(L);
            if constexpr (MODE != 2 && f_ >= 0) fetch(LATE, f_);
            if constexpr (MODE != 2 && r_ >= 0) read_scales(sc_next, r_);
            if constexpr (MODE != 2 && t_ >= 0) settle_scales(FMT ? t_ >> 2 : settle_set(t_ >> 2), t_ & 3, MODE == 1);
            if (!RAG && STEADY && L == 0) dma16(sc_dst, svoff + sc_off, sc_src);
            if (RAG && STEADY && L == 0) {
                rag_store((s + 1) / BATCH + 1, (s + 1) & 3, par, sp[4]);
                sp[4] = rag_load(cur, (s + 2) / BATCH + 1, (s + 2) & 3);
            }
            if constexpr (RAG && MODE == 1 && w_ >= 0) sp[w_] = rag_load(nxt, w_ / 4, w_ & 3);
            if constexpr (RAG && MODE == 2 && w_ >= 0) rag_store(w_ / 4, w_ & 3, par_nxt, sp[w_]);
            if (RAG && MODE == 2 && L == LATE_GAPS - 1) sp[4] = rag_load(nxt, 1, 1);
            if constexpr (STEADY && d_ >= 0) issue_load(IC<d_ < 0 ? 0 : d_>{}, no_force{});
            if constexpr (MODE == 1 && d_ >= 0) issue_load(IC<d_ < 0 ? 0 : d_>{}, force_m0{});
            if constexpr (!RAG && MODE == 1 && w_ >= 0 && w_ < (NJ == 4 ? 4 : 3)) issue_scales(nxt, 0, w_, par_nxt);
            if (!RAG && MODE == 2 && L == 1) issue_scales(nxt, 1, 0, par_nxt);
        };
#define MXFP4_K0(G)                                                                              \
        {                                                                                        \
            constexpr int f_ = FMT ? MXFP4_AT(G, 1, 2, 8) : NJ == 4 ? MXFP4_AT(G, 2, 4, 8) : MXFP4_AT(G, 1, 2, 6); \
            constexpr int d_ = FMT ? MXFP4_AT(G, 0, 2, 4) : NJ == 4 ? MXFP4_AT(G, 0, 4, 4) : MXFP4_AT(G, 0, 2, 4); \
            constexpr int a_ = FMT ? MXFP4_AT(G, 8, 2, 4) : NJ == 4 ? MXFP4_AT(G, 3, 2, 8) : MXFP4_AT(G, 8, 1, 6); \
            if constexpr (f_ >= 0) fetch(0, f_);                                                 \
            if constexpr (a_ >= 0) age_scales(a_);                                               \
            if constexpr (d_ >= 0) issue_load(IC<LOADS_LATE + (d_ < 0 ? 0 : d_)>{}, no_force{}); \
        }                                                                                        \
        MXFP4_SLOT_MMA(0, G, MODE) MXFP4_PIN()
        MXFP4_32(MXFP4_K0)
#undef MXFP4_K0
#define MXFP4_K1(G)                                                                              \
        {                                                                                        \
            constexpr int f_ = FMT ? MXFP4_AT(G, 0, 2, 8) : NJ == 4 ? MXFP4_AT(G, 0, 3, 10) : MXFP4_AT(G, 0, 2, 8); \
            constexpr int n_ = !FMT && NJ == 4 ? MXFP4_AT(G, 1, 4, 8) : MXFP4_AT(G, 1, 2, 8);     \
            if constexpr (f_ >= 0) fetch(1, f_);                                                 \
            if constexpr (n_ >= 0) step(n_);                                                     \
        }                                                                                        \
        if (!FMT && (G) == GAPS - 2) other_buffer(ra[0]); /* (K-step 0's fragments have all been fetched) */ \
        if (!FMT && (G) == GAPS - 1) other_buffer(rb[0]);                                        \
        MXFP4_SLOT_MMA(1, G, MODE) MXFP4_PIN()
        MXFP4_32(MXFP4_K1)
#undef MXFP4_K1
#define MXFP4_K2(G)                                                                              \
        if constexpr (!FMT && (G) < 2 * 4 && (G) % 2 == 0) fetch(2, (G) / 2); /* (early: the barrier waits for them) */ \
        if (FMT && (G) < 2) other_buffer(ra[(G) & 1]); /* (the stage's fragments have all been fetched) */ \
        if (FMT && (G) >= 2 && (G) < 4) other_buffer(rb[(G) & 1]);                               \
        if constexpr ((G) == BAR) {                                                              \
            /* every wave has fetched its last fragments of this buffer, and this wave's loads of the next stage have landed: */ \
            /* after the barrier the buffer may be refilled and the other read */                \
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                                     \
            __syncthreads();                                                                     \
        }                                                                                        \
        if constexpr ((G) >= BAR && (G) < GAPS) late(IC<((G) >= BAR ? (G) - BAR : 0)>{});        \
        MXFP4_SLOT_MMA(2, G, MODE) MXFP4_PIN()
        MXFP4_32(MXFP4_K2)
#undef MXFP4_K2
#define MXFP4_K3(G)                                                                              \
        if constexpr ((G) < GAPS) late(IC<GAPS - BAR + (G)>{});                                  \
        if (!FMT && (G) == GAPS - 2) other_buffer(ra[1]);                                        \
        if (!FMT && (G) == GAPS - 1) other_buffer(rb[1]);                                        \
        MXFP4_SLOT_MMA(3, G, MODE) MXFP4_PIN()
        MXFP4_32(MXFP4_K3)
#undef MXFP4_K3
    };
    using mode_main = std::integral_constant<int, 0>;
    using mode_penult = std::integral_constant<int, 1>;
    using mode_last = std::integral_constant<int, 2>;
    using mode_first = std::integral_constant<int, 3>;

    // ---- first tile: fill the pipeline --------------------------------------------------------
    // all of stage 0, scale batch 0 and the first load of batch 1
    TileSrc cur = tile_src(lw);
    set_load(cur, 0);
#define MXFP4_FILL(N) if constexpr ((N) < NLOADS) issue_load(IC<((N) < NLOADS ? (N) : 0)>{}, no_force{});
    MXFP4_16(MXFP4_FILL)
#undef MXFP4_FILL
    if constexpr (RAG) {
#pragma unroll
        for (int j = 0; j < 5; ++j) sp[j] = rag_load(cur, j / 4, j & 3);
#pragma unroll
        for (int j = 0; j < 5; ++j) rag_store(j / 4, j & 3, 0, sp[j]);
        sp[4] = rag_load(cur, 1, 1);
    } else {
#pragma unroll
        for (int j = 0; j < (NJ == 4 ? 4 : 3); ++j) issue_scales(cur, 0, j, 0);
        issue_scales(cur, 1, 0, 0);
    }
    int par = 0;
    const int b_last = (nstages - 1) / BATCH;

    for (int lloc = lw; lloc < count_x; lloc += nwg_x) {
        const int par_nxt = (b_last ^ par ^ 1) & 1;
        // the tile after this one; after the last tile the hand-over loads simply fetch that tile's
        // first stage again into buffers that are idle by then (no branches in the stage bodies)
        const TileSrc nxt = (lloc + nwg_x < count_x) ? tile_src(lloc + nwg_x) : cur;
        // entering a tile: its stage 0 and first scale batch have landed (first tile: wait for them
        // here); after the barrier start most of stage 1's loads (LOADS_LATE) and fetch the first fragments
        if (lloc == lw) asm volatile("s_waitcnt vmcnt(1)" ::: "memory");  // (later tiles waited before the epilogue)
        __syncthreads();
        set_load(cur, 1);
        ld_buf ^= STAGE_BYTES;
#define MXFP4_FILL(N) if constexpr ((N) < LOADS_LATE) issue_load(IC<((N) < LOADS_LATE ? (N) : 0)>{}, no_force{});
        MXFP4_16(MXFP4_FILL)
#undef MXFP4_FILL
#pragma unroll
        for (int n = 0; n < (FMT ? 16 : NB + 2); ++n) fetch(LATE, n);
#pragma unroll
        for (int n = 0; n < (NJ == 4 ? 4 : 3); ++n) read_scales((uint32_t)(par << 14), n);
#pragma unroll
        for (int t = 0; t < 4 * SETS; ++t) settle_scales(FMT ? t >> 2 : settle_set(t >> 2), t & 3, false);
        __builtin_amdgcn_sched_barrier(0);

        stage(cur, nxt, par, par_nxt, 0, mode_first{});
        for (int s = 1; s + 2 < nstages; ++s) stage(cur, nxt, par, par_nxt, s, mode_main{});
        stage(cur, nxt, par, par_nxt, nstages - 2, mode_penult{});
        stage(cur, nxt, par, par_nxt, nstages - 1, mode_last{});
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");  // (the last sums are written 19 clocks' worth of instructions after they are issued)
        __builtin_amdgcn_sched_barrier(0);
        // the next tile's stage 0 and scale batch 0 have been on their way for at least two K-steps: make
        // sure they have landed now, before any store is issued (only the one scale load of batch 1 issued
        // a moment ago may stay out), so that nothing later has to wait for the stores to drain
        asm volatile("s_waitcnt vmcnt(1)" ::: "memory");

        // ---- epilogue ---------------------------------------------------------------------------
        // The output is stored non-temporally: it is not read again here, and written the ordinary way it
        // pushes the operands of the kernels that follow (the next quantisers, the next GEMM) out of the
        // last-level cache -- measured on the 8B fused-QKV layer: 10 % of a whole forward + backward step.
        // A lane owns row fr of each 16-row group and, per 16-column group, columns 4*fg + {0..3}.
        // The last stage's buffer is free (all waves passed the last barrier; the other one may already hold
        // the next tile's stage 0): each wave transposes its sub-tile through its own 16 KiB slice of it, 64
        // (bf16) or 32 (fp32) rows at a time, and writes whole 256- / 512-byte row segments.  Rows are
        // stored unpadded; 16-byte chunk c of row r sits at chunk c ^ (r & 15), which keeps both the 8/16-byte writes and the 16-byte
        // reads conflict-free.
        uint8_t *epi = smem + ((((nstages - 1) & 1) ^ bp) ? STAGE_BYTES : 0) + wave * 16384;
        const int64_t row0 = cur.m0 + wm * 128, col0 = cur.n0 + wn * (32 * NJ);
        // RAG: a tile that was moved back stores only what is its own: the others' pieces get an offset beyond the buffer,
        // which the hardware drops (a branch per store costs the registers: the sums then no longer fit).  row, col: within
        // the wave's sub-tile.
        constexpr int ESIZE = OUT_FP32 ? 4 : 2;
        __amdgpu_buffer_rsrc_t rsrc;
        if constexpr (RAG)
            rsrc = __builtin_amdgcn_make_buffer_rsrc(static_cast<uint8_t *>(out) + (row0 * ld + col0) * ESIZE, 0, 0x7FFFFFFF,
                                                     0x00020000);
        auto rag_offset = [&](int row, int col) {
            const bool mine = wm * 128 + row >= cur.dm && wn * (32 * NJ) + col >= cur.dn;
            return mine ? (row * (int)ld + col) * ESIZE : (int)0x80000000u;
        };
        auto rag_put = [&](int row, int col, auto v) {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), rsrc, rag_offset(row, col), 0, 2 /* nt */);
        };
        // ACC: the values added to are loaded eight at a time (whole narrow tiles: a batch ahead).  Loaded one by one in front of their
        // stores, which the compiler must keep in that order, they were 32 or 64 round trips to memory per tile.  fp32 added to, us, before /
        // now: 6144 x 4096 x 8192 131 / 120, 28672 x 4096 x 8192 690 / 515, 4096 x 14336 x 4096 233 / 165, 1024 x 4096 x 8192 (narrow) 42.1 /
        // 33.7; moved back 10000 x 8576 x 1760 344 / 210, 4320 x 1440 x 2080 27.9 / 21.7; MXFP8 4096 x 4096 x 2048 52.3 / 44.2.
        constexpr int RPS = NJ == 2 ? 4 : 2;  // fp32 rows per store instruction
        constexpr bool AHEAD = ACC && !RAG && NJ == 2;
        v4f prev[AHEAD ? 2 : 1][8];
        auto load_prev = [&](int first, int set) {
            if (first >= (NJ == 2 ? 32 : 64)) return;
            const float *from = reinterpret_cast<const float *>(out) + (row0 + first * RPS + lane / (64 / RPS)) * ld + col0 + lane % (64 / RPS) * 4;
#pragma unroll
            for (int u = 0; u < 8; ++u) prev[set][u] = *reinterpret_cast<const v4f *>(from + (int64_t)(u * RPS) * ld);
        };
        auto rag_put8 = [&](int row, int col, const v4f (&buf)[8]) {  // RAG: rows row + RPS u
            int off[8];
            v4f old[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                off[u] = rag_offset(row + RPS * u, col);
                if constexpr (ACC) old[u] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[u], 0, 0));
            }
            __builtin_amdgcn_sched_barrier(0);  // (without it the offsets of later batches are worked out here and the sums spill)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v4f v = buf[u];
                if constexpr (ACC) v += old[u];
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), rsrc, off[u], 0, 2 /* nt */);
            }
        };
        if constexpr (AHEAD) load_prev(0, 0);
        if constexpr (NJ == 2 && !OUT_FP32) {
            // Narrow tile, bf16: the wave's 128 rows x 64 columns are 16 KiB, one pass.  A row is 8 chunks of 16
            // bytes; chunk c of row r sits at position c ^ ((r >> 1) & 7): the 8-byte writes of a quarter wave
            // (16 rows, one chunk) and the 16-byte reads (2 rows x 8 chunks) then cover all banks evenly.
#pragma unroll
            for (int i = 0; i < 8; ++i) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = i * 16 + fr, c = j * 2 + (fg >> 1);
                    uint2 pk;
                    pk.x = pack_bf16(acc[i][j][0], acc[i][j][1]);
                    pk.y = pack_bf16(acc[i][j][2], acc[i][j][3]);
                    *reinterpret_cast<uint2 *>(epi + r * 128 + ((c ^ ((r >> 1) & 7)) << 4) + ((fg & 1) << 3)) = pk;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // 8 lanes x 16 bytes = one 128-byte row segment; 8 rows per instruction
            int rl = lane >> 3, ch = lane & 7;
            if (RAG) asm volatile("" : "+v"(rl), "+v"(ch));  // (else every offset is worked out ahead of the tile loop)
            uint16_t *obase = reinterpret_cast<uint16_t *>(out) + (row0 + rl) * ld + col0 + ch * 8;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4i buf[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int r = (8 * h + u) * 8 + rl;
                    buf[u] = *reinterpret_cast<const v4i *>(epi + r * 128 + ((ch ^ ((r >> 1) & 7)) << 4));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if constexpr (RAG) rag_put((8 * h + u) * 8 + rl, ch * 8, buf[u]);
                    else __builtin_nontemporal_store(buf[u], reinterpret_cast<v4i *>(obase + (int64_t)((8 * h + u) * 8) * ld));
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if constexpr (NJ == 2) {
            // Narrow tile, fp32: 128 rows x 256 bytes in two passes of 64 rows; chunk c (4 columns) of row r at
            // position c ^ (r & 15)
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
                for (int ii = 0; ii < 4; ++ii) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int r = ii * 16 + fr, c = j * 4 + fg;
                        *reinterpret_cast<v4f *>(epi + r * 256 + ((c ^ (r & 15)) << 4)) = acc[4 * pass + ii][j];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                // 16 lanes x 16 bytes = one 256-byte row segment; 4 rows per instruction
                int rl = lane >> 4, ch = lane & 15;
                if (RAG) asm volatile("" : "+v"(rl), "+v"(ch));  // (else every offset is worked out ahead of the tile loop)
                float *obase = reinterpret_cast<float *>(out) + (row0 + pass * 64 + rl) * ld + col0 + ch * 4;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v4f buf[8];
                    if constexpr (ACC && !RAG) load_prev(8 * (2 * pass + h + (AHEAD ? 1 : 0)), AHEAD ? 1 - h : 0);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int r = (8 * h + u) * 4 + rl;
                        buf[u] = *reinterpret_cast<const v4f *>(epi + r * 256 + ((ch ^ (r & 15)) << 4));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (RAG) {
                        rag_put8(pass * 64 + 8 * h * 4 + rl, ch * 4, buf);
                    } else {
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            v4f v = buf[u];
                            if constexpr (ACC) v += prev[AHEAD ? h : 0][u];
                            __builtin_nontemporal_store(v, reinterpret_cast<v4f *>(obase + (int64_t)((8 * h + u) * 4) * ld));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else if constexpr (!OUT_FP32) {
#pragma unroll
            for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
                for (int ii = 0; ii < 4; ++ii)
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int i = 4 * pass + ii;
                        const int r = ii * 16 + fr, c = j * 2 + (fg >> 1);
                        uint2 pk;
                        pk.x = pack_bf16(acc[i][j][0], acc[i][j][1]);
                        pk.y = pack_bf16(acc[i][j][2], acc[i][j][3]);
                        *reinterpret_cast<uint2 *>(epi + r * 256 + ((c ^ (r & 15)) << 4) + ((fg & 1) << 3)) = pk;
                        if (j & 4) __builtin_amdgcn_sched_barrier(0);
                    }
                // 16 lanes x 16 bytes = one 256-byte row segment; 4 rows per instruction.  Eight LDS reads are
                // issued before the first store needs its data, so their latencies overlap; the row pointer
                // is one per-lane base plus a scalar multiple of the leading dimension.
                int rl = lane >> 4, ch = lane & 15;
                if (RAG) asm volatile("" : "+v"(rl), "+v"(ch));  // (else every offset is worked out ahead of the tile loop)
                uint32_t roff[4];  // LDS offset of this lane's chunk in rows rl, 4 + rl, 8 + rl, 12 + rl
#pragma unroll
                for (int k = 0; k < 4; ++k) roff[k] = (uint32_t)((4 * k + rl) * 256 + ((ch ^ (4 * k + rl)) << 4));
                uint16_t *obase = reinterpret_cast<uint16_t *>(out) + (row0 + pass * 64 + rl) * ld + col0 + ch * 8;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v4i buf[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int r4 = (8 * h + u) * 4;
                        buf[u] = *reinterpret_cast<const v4i *>(epi + (r4 & ~15) * 256 + roff[(r4 >> 2) & 3]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int r4 = (8 * h + u) * 4;
                        if constexpr (RAG) rag_put(pass * 64 + r4 + rl, ch * 8, buf[u]);
                        else __builtin_nontemporal_store(buf[u], reinterpret_cast<v4i *>(obase + (int64_t)r4 * ld));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
#pragma unroll
            for (int pass = 0; pass < 4; ++pass) {
#pragma unroll
                for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int r = ii * 16 + fr, c = j * 4 + fg;
                        *reinterpret_cast<v4f *>(epi + r * 512 + ((c ^ r) << 4)) = acc[2 * pass + ii][j];
                        if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                    }
                // 32 lanes x 16 bytes = one 512-byte row segment; 2 rows per instruction; reads batched by
                // eight as above
                int rl = lane >> 5, ch = lane & 31;
                if (RAG) asm volatile("" : "+v"(rl), "+v"(ch));  // (else every offset is worked out ahead of the tile loop)
                float *obase = reinterpret_cast<float *>(out) + (row0 + pass * 32 + rl) * ld + col0 + ch * 4;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v4f buf[8];
                    if constexpr (ACC && !RAG) load_prev(8 * (2 * pass + h + (AHEAD ? 1 : 0)), AHEAD ? 1 - h : 0);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int r = (8 * h + u) * 2 + rl;
                        buf[u] = *reinterpret_cast<const v4f *>(epi + r * 512 + ((ch ^ r) << 4));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (RAG) {
                        rag_put8(pass * 32 + 8 * h * 2 + rl, ch * 4, buf);
                    } else {
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            v4f v = buf[u];
                            if constexpr (ACC) v += prev[AHEAD ? h : 0][u];
                            __builtin_nontemporal_store(v, reinterpret_cast<v4f *>(obase + (int64_t)((8 * h + u) * 2) * ld));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // (the barrier at the top of the loop keeps the next tile's loads out of that buffer until
        // every wave is done reading its slice)
        cur = nxt;
        par = par_nxt;
        bp ^= nstages & 1;
    }
    // nothing may still be writing this workgroup's LDS when it retires
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#undef MXFP4_MFMA
#undef MXFP4_SLOT_MMA
#undef MXFP4_PIN
#undef MXFP4_AT
#undef MXFP4_32
#undef MXFP4_16
}

struct TileGemm {
    const uint8_t *aq, *as, *bq, *bs;
    int64_t C;
    void *out;
    int64_t ld;
    int tiles_m, tiles_n;
};

template <bool OUT_FP32, bool ACC, int FMT, int NJ>
__global__ __launch_bounds__(256, 1) void gemm_tile_kernel(const TileGemm p)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS_BYTES];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    gemm_tile_body<OUT_FP32, ACC, FMT, NJ>(p.aq, p.as, p.bq, p.bs, p.C, p.out, p.ld, p.tiles_m, p.tiles_n,
                                           blockIdx.x, gridDim.x, smem, lds0);
}

// One launch for a product whose last round of 256 x 256 tiles is at most half full: every workgroup first walks
// the whole rounds (tiles 0 .. t_main-1 of the sequence) on 256 x 256 tiles, then the remaining tiles are worked on
// as twice as many 256 x 128 tiles, one per workgroup, so that the compute units that would idle in the last round
// take half of it.  (Nothing is prefetched across the two phases: the second one fills its pipeline again.)
template <bool OUT_FP32, bool ACC>
__global__ __launch_bounds__(256, 1) void gemm_tile_tail_kernel(const TileGemm p, const int t_main)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS_BYTES];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    gemm_tile_body<OUT_FP32, ACC, 0, 4>(p.aq, p.as, p.bq, p.bs, p.C, p.out, p.ld, p.tiles_m, p.tiles_n, blockIdx.x,
                                        gridDim.x, smem, lds0, 0, t_main);
    __syncthreads();  // (every wave is done with the LDS of the first phase)
    gemm_tile_body<OUT_FP32, ACC, 0, 2, true>(p.aq, p.as, p.bq, p.bs, p.C, p.out, p.ld, p.tiles_m, p.tiles_n,
                                              blockIdx.x, gridDim.x, smem, lds0, t_main, p.tiles_m * p.tiles_n);
}

// Two independent products of which one (pn) has at most one 256 x 128 tile for each of some compute units and the other
// (pw) many 256 x 256 ones (Wgrad and Dgrad of a k or v projection): on every XCD the first n1 of the 32 workgroups take
// one tile of pn each and then walk tiles 0 .. cut-1 of pw, the others walk the rest of pw.  One after the other, half the
// chip idled under pn: the step of an 8B
// k projection (Dgrad 8192 x 4096 x 1024, Wgrad 1024 x 4096 x 8192) went from 114.1 to 104.9 us.
template <bool OUTN, bool ACCN, bool OUTW, bool ACCW>
__global__ __launch_bounds__(256, 1) void gemm_tile_mix_kernel(const TileGemm pn, const TileGemm pw, const int n1,
                                                               const int cut)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS_BYTES];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int xcd = blockIdx.x & 7, lw = blockIdx.x >> 3;
    const bool first = lw < n1;
    if (first) {
        gemm_tile_body<OUTN, ACCN, 0, 2>(pn.aq, pn.as, pn.bq, pn.bs, pn.C, pn.out, pn.ld, pn.tiles_m, pn.tiles_n,
                                         lw * 8 + xcd, (uint32_t)n1 * 8, smem, lds0);
        __syncthreads();  // (every wave is done with the LDS of the first product)
    }
    gemm_tile_body<OUTW, ACCW, 0, 4>(pw.aq, pw.as, pw.bq, pw.bs, pw.C, pw.out, pw.ld, pw.tiles_m, pw.tiles_n,
                                     (first ? lw : lw - n1) * 8 + xcd, (uint32_t)(first ? n1 : 32 - n1) * 8, smem, lds0,
                                     first ? 0 : cut, first ? cut : pw.tiles_m * pw.tiles_n);
}

// Ragged sizes on the same tiles: t_main tiles of the sequence on 256 x 256, then (MXFP4) the rest in halves.  Measured,
// bf16 output, gemm_edge_kernel / this one: 8192 x 6144 x 4064 181 / 112 us (3.7 PFLOP/s; MXFP8 273 / 188), 4096 x 4096 x 4000
// 58 / 39; 4010 x 6144 x 4096 54 us (with 32 x 32 x 64 instructions 116, 196, 40.4 and 55.2).
template <bool OUT_FP32, bool ACC, int FMT>
__global__ __launch_bounds__(256, 1) void gemm_tile_rag_kernel(const TileGemm p, const int64_t Ra, const int64_t Rb,
                                                               const int t_main)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS_BYTES];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    gemm_tile_body<OUT_FP32, ACC, FMT, 4, false, true>(p.aq, p.as, p.bq, p.bs, p.C, p.out, p.ld, p.tiles_m, p.tiles_n,
                                                       blockIdx.x, gridDim.x, smem, lds0, 0, t_main, Ra, Rb);
    if constexpr (FMT == 0) {
        if (t_main == p.tiles_m * p.tiles_n) return;
        __syncthreads();  // (every wave is done with the LDS of the first phase)
        gemm_tile_body<OUT_FP32, ACC, 0, 2, true, true>(p.aq, p.as, p.bq, p.bs, p.C, p.out, p.ld, p.tiles_m, p.tiles_n,
                                                        blockIdx.x, gridDim.x, smem, lds0, t_main,
                                                        p.tiles_m * p.tiles_n, Ra, Rb);
    }
}

// The same for two independent products of ragged sizes (Dgrad and Wgrad of a layer whose widths are in no whole tiles): as in
// gemm_tile_pair_kernel the first n0 of every XCD's 32 workgroups work on p0, the others on p1; each product is cut into 256 x 256 tiles or,
// where that fills its share of the chip better, into 256 x 128 ones (narrow0, narrow1).  Side by side on 128 x 256 tiles of
// gemm_edge_kernel, or one after the other with half the chip idle, such a pair took 1.04 to 1.42 times as long.  us, before / now, layers of
// M x N x K: 2080 x 4320 x 1440 36.4 / 31.8, 4128 x 4320 x 4064 138 / 116, 1760 x 3584 x 2400 34.0 / 27.7, 1728 x 10112 x 3008 105 / 84; dW added
// to: 2592 x 5344 x 1280 46.5 / 36.7, 2336 x 2336 x 2336 40.2 / 31.6, 4320 x 2016 x 3264 67.1 / 47.2.
template <bool OUT0, bool ACC1>
__global__ __launch_bounds__(256, 1) void gemm_tile_rag_pair_kernel(const TileGemm p0, const int64_t Ra0, const int64_t Rb0, const int narrow0,
                                                                    const TileGemm p1, const int64_t Ra1, const int64_t Rb1,
                                                                    const int narrow1, const int n0)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS_BYTES];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int xcd = blockIdx.x & 7, lw = blockIdx.x >> 3;
    if (lw < n0) {
        const int T = p0.tiles_m * p0.tiles_n;
        if (narrow0)
            gemm_tile_body<OUT0, false, 0, 2, true, true>(p0.aq, p0.as, p0.bq, p0.bs, p0.C, p0.out, p0.ld, p0.tiles_m, p0.tiles_n,
                                                          lw * 8 + xcd, (uint32_t)n0 * 8, smem, lds0, 0, T, Ra0, Rb0);
        else
            gemm_tile_body<OUT0, false, 0, 4, false, true>(p0.aq, p0.as, p0.bq, p0.bs, p0.C, p0.out, p0.ld, p0.tiles_m, p0.tiles_n,
                                                           lw * 8 + xcd, (uint32_t)n0 * 8, smem, lds0, 0, T, Ra0, Rb0);
    } else {
        const int T = p1.tiles_m * p1.tiles_n;
        if (narrow1)
            gemm_tile_body<true, ACC1, 0, 2, true, true>(p1.aq, p1.as, p1.bq, p1.bs, p1.C, p1.out, p1.ld, p1.tiles_m, p1.tiles_n,
                                                         (lw - n0) * 8 + xcd, (uint32_t)(32 - n0) * 8, smem, lds0, 0, T, Ra1, Rb1);
        else
            gemm_tile_body<true, ACC1, 0, 4, false, true>(p1.aq, p1.as, p1.bq, p1.bs, p1.C, p1.out, p1.ld, p1.tiles_m, p1.tiles_n,
                                                          (lw - n0) * 8 + xcd, (uint32_t)(32 - n0) * 8, smem, lds0, 0, T, Ra1, Rb1);
    }
}

// Two independent GEMMs in one launch of 256 workgroups (Dgrad and Wgrad of one layer): on every XCD the
// first n0 of its 32 workgroups work on p0, the others on p1, each set walking its own problem's tiles.
// The CUs are split in proportion to the work, so both problems end on full rounds of tiles.  Measured on
// the 8B shapes the launch takes about 5 % less than the two GEMMs one after the other (173-180 against
// 181-195 us): one dispatch gap and one pipeline fill less, no part-filled round, and the two problems' tiles
// have different lengths, so that their output bursts fall at different times.  It is not more: with half
// the chip idle in a partly filled last round the busy half clocks higher under the power cap, and here each
// XCD's L2 holds panels of two problems (22 % more traffic beyond L2).
// FMT0, FMT1: element format of each problem's operands (0 = E2M1, 1 = E4M3), as in gemm_tile_kernel.
template <bool OUT0, bool OUT1, bool ACC1, int FMT0, int FMT1>
__global__ __launch_bounds__(256, 1) void gemm_tile_pair_kernel(const TileGemm p0, const TileGemm p1, const int n0)
{
    __shared__ __attribute__((aligned(1024))) uint8_t smem[LDS_BYTES];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const uint32_t xcd = blockIdx.x & 7, lw = blockIdx.x >> 3;
    if (lw < (uint32_t)n0)
        gemm_tile_body<OUT0, false, FMT0, 4>(p0.aq, p0.as, p0.bq, p0.bs, p0.C, p0.out, p0.ld, p0.tiles_m, p0.tiles_n,
                                             lw * 8 + xcd, (uint32_t)n0 * 8, smem, lds0);
    else
        gemm_tile_body<OUT1, ACC1, FMT1, 4>(p1.aq, p1.as, p1.bq, p1.bs, p1.C, p1.out, p1.ld, p1.tiles_m, p1.tiles_n,
                                            (lw - n0) * 8 + xcd, (uint32_t)(32 - n0) * 8, smem, lds0);
}

// ---- ragged-shape kernel: any row and column counts, any C % 32 == 0 --------------------------
// 2 x NWN waves on a (64 WM) x (32 WN NWN) output tile, V_MFMA_SCALE_F32_32X32X64_F8F6F4, WM x WN of them per wave and
// K-step.  It is bound by how fast operands reach the matrix unit: the kernel it took over from read every fragment
// straight from global memory, 16 rows x 64 bytes per instruction and each row by two waves, with nothing in flight
// while it multiplied.  Here codes go global -> LDS in whole 128-byte row pieces (one stage = 128 bytes of every row,
// NBUF stage buffers), each row piece once per workgroup, under the swizzle of the tiled kernel above.
// What makes it any-shape:
//   * rows beyond the matrix are clamped to the last one (their results are dropped by the store);
//   * a 16-byte chunk beyond the end of a row is clamped to the row's last chunk, and the scale bytes of the blocks
//     beyond C/32 are 0 in LDS for both operands: every product under them is below 2^-254 * 2^24, which is 0 in fp32,
//     so the last stage runs the same code as the others;
//   * scale rows are C/32 bytes apart, at any alignment: they come through registers (16-byte loads, shifted and
//     masked at a row's ragged end) into LDS, 32 bytes per row (1024 elements of K) at a time.
// FMT as in gemm_tile_body.  Built as 64 x 64 (4 stage buffers, 68 KiB of LDS, two workgroups per CU), 128 x 64 (3, 78 KiB,
// two) and 128 x 256 tiles (8 waves, 3, 156 KiB; with two stage buffers 8192 x 6112 x 4064 took 185 us, with three 173);
// 128 x 128 tiles on 4 waves were never the fastest, 256 x 256 tiles on 8 waves were slower for MXFP4 (210 against 156 us).
// What bounds it now: at 8192 x 6144 x 4096 (153 us, 2.7 PFLOP/s, against 89 us of the tiled kernel) LDS traffic, 176 KiB
// per 128 x 256 stage against 1024 clocks of matrix instructions; rows that are not whole cache lines apart cost another
// 20 % (C = 4064: 181 us), because every 128-byte row piece then takes two line requests.
// Measured back to back in a graph, bf16 output, the any-shape kernel / the fastest tile of this one: MXFP4 8192 x 6144 x 4064
// 902 / 181 us (now on moved-back tiles, 112), 16000 x 1000 x 3008 238 / 47, 2080 x 4320 x 1440 69 / 21, 2048 x 3072 x 768
// 33 / 9, 200 x 4096 x 4096 31 / 8.5, 24 x 6144 x 4096 23.5 / 7.9 (now on 32 x 32 tiles, 5.6); MXFP8 8192 x 6144 x 4064
// 1335 / 273 (on moved-back tiles 188), 200 x 4096 x 4096 45.5 / 11.9 us.
template <int WM, int WN, int NWN, int NBUF>
struct EdgeTile {
    static constexpr int WAVES = 2 * NWN, TM = 64 * WM, TN = 32 * WN * NWN, ROWS = TM + TN;
    static constexpr int STAGE = ROWS * 128;          // bytes of codes per stage
    static constexpr int NL = ROWS / 8 / WAVES;              // direct-to-LDS loads per wave and stage
    static constexpr int OFF_S = NBUF * STAGE;
    static constexpr int LDS = OFF_S + ROWS * 32;
};

struct EdgeGemm {
    const uint8_t *aq, *as, *bq, *bs;
    int64_t Ra, Rb, C;
    void *out;
    int64_t ld;
    int tiles_m, tiles_n;
    int out_fp32, accumulate;
    int vec;  // bits: 1 four consecutive outputs may be stored at once, 2 sixteen bytes of them, 4 rows are whole cache lines,
              // 8 rows are whole 4 bytes (but not 16)
};

// Whether workgroup `bid` has a tile (the grid is padded to whole rows of 8) is asked apart from which one: as one function with both
// answers the compiler loads the operands' pointers only behind the divisions, 0.2 us later (200 x 4096 x 4096 8.42 us, 8.24 like this).
__device__ __forceinline__ bool edge_has_tile(const EdgeGemm &p, uint32_t bid)
{
    const int T = p.tiles_m * p.tiles_n;
    return (int)(bid >> 3) < (T >> 3) + ((int)(bid & 7) < (T & 7) ? 1 : 0);
}
// The tile (tm x tn) of workgroup `bid`, which has one: each XCD (workgroup id mod 8) takes a contiguous run of the tile sequence, which walks the grid in
// groups of GROUP_M tile rows (as the tiled kernel does).
__device__ __forceinline__ void edge_tile(const EdgeGemm &p, uint32_t bid, int tm, int tn, int64_t &m0, int64_t &n0)
{
    const int T = p.tiles_m * p.tiles_n, xcd = bid & 7, per = T >> 3, rem = T & 7;
    const int L = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + (int)(bid >> 3);
    const int span = GROUP_M * p.tiles_n, grp = L / span, first = grp * GROUP_M, in = L - grp * span;
    const int gm = p.tiles_m - first < GROUP_M ? p.tiles_m - first : GROUP_M;
    // (uniform, but the division ran in the vector unit: put them where the loads want their base)
    m0 = (int64_t)__builtin_amdgcn_readfirstlane(first + in % gm) * tm;
    n0 = (int64_t)__builtin_amdgcn_readfirstlane(in / gm) * tn;
}

// four consecutive outputs of one row from column col on, at once (whole: what they are added to is in v already) or as many of them as
// are left
template <bool ACC>
__device__ __forceinline__ void store4(const EdgeGemm &p, int64_t row, int64_t col, int64_t left, bool whole, const v4f v)
{
    if (p.out_fp32) {
        float *o = reinterpret_cast<float *>(p.out) + row * p.ld + col;
        if (whole) {
            __builtin_nontemporal_store(v, reinterpret_cast<v4f *>(o));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < left) o[e] = ACC && p.accumulate ? (o[e] + v[e]) : v[e];
        }
    } else {
        uint16_t *o = reinterpret_cast<uint16_t *>(p.out) + row * p.ld + col;
        const uint32_t lo = pack_bf16(v[0], v[1]), hi = pack_bf16(v[2], v[3]);
        if (whole) {
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            __builtin_nontemporal_store((u32x2){lo, hi}, reinterpret_cast<u32x2 *>(o));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e < left) o[e] = (uint16_t)((e & 2 ? hi : lo) >> (16 * (e & 1)));
        }
    }
}

// A launch may carry two independent problems: workgroups 0 .. groups0-1 (a multiple of 8) work on p0, the others on p1.
// ACC: a product of the launch is added to its output.
template <int FMT, int WM, int WN, int NWN, int NBUF, bool ACC>
__global__ __launch_bounds__(128 * NWN, 2) void gemm_edge_kernel(const EdgeGemm p0, const EdgeGemm p1, const uint32_t groups0)
{
    const bool second = blockIdx.x >= groups0;  // uniform
    const EdgeGemm p = second ? p1 : p0;
    const uint32_t bid = blockIdx.x - (second ? groups0 : 0u);
    using Tile = EdgeTile<WM, WN, NWN, NBUF>;
    constexpr int TM = Tile::TM, TN = Tile::TN, NL = Tile::NL, ROWS = Tile::ROWS, WAVES = Tile::WAVES;
    constexpr int NLA = TM / 8 / WAVES;  // loads of A among a wave's NL
    constexpr int BATCH = FMT ? 8 : 4;  // stages per scale batch
    __shared__ __attribute__((aligned(1024))) uint8_t smem[Tile::LDS];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / NWN, wn = wave % NWN;

    int64_t m0, n0;
    if (!edge_has_tile(p, bid)) return;
    edge_tile(p, bid, TM, TN, m0, n0);

    const int64_t rowbytes = FMT ? p.C : (p.C >> 1);
    const int nkb = (int)(p.C >> 5);
    const int nstages = (int)((rowbytes + 127) >> 7);
    const int nbatches = (nkb + 31) >> 5;
    const uint8_t *abase = p.aq + m0 * rowbytes, *bbase = p.bq + n0 * rowbytes;

    // direct-to-LDS loads: load n of wave w moves the 8-row group WAVES n + w (A's rows, then B's)
    const int drr = lane >> 3, chunk = ((lane & 7) ^ drr ^ (wave & 1)) << 4;
    uint32_t roff[NL];
#pragma unroll
    for (int n = 0; n < NL; ++n) {
        const bool isb = n >= NLA;
        const int64_t r0 = isb ? n0 : m0, R = isb ? p.Rb : p.Ra;
        const int64_t want = (int64_t)((n - (isb ? NLA : 0)) * WAVES + wave) * 8 + drr, last = R - 1 - r0;
        roff[n] = (uint32_t)((want < last ? want : last) * rowbytes);
    }
    auto issue = [&](int s, int to) {
        const uint32_t at = (uint32_t)s * 128u + (uint32_t)chunk, end = (uint32_t)rowbytes - 16u;
        const uint32_t koff = at < end ? at : end;
        const uint32_t dst = lds0 + (uint32_t)to * Tile::STAGE + (uint32_t)wave * 1024u;
#pragma unroll
        for (int n = 0; n < NL; ++n) dma16(dst + n * (WAVES * 1024u), roff[n] + koff, n >= NLA ? bbase : abase);
    };

    // scale bytes: piece j of this thread = 16 bytes (half (tid * NP + j) & 1 of its row's 32) of a batch
    constexpr int NP = (ROWS * 2 + 64 * WAVES - 1) / (64 * WAVES);
    uint4 piece[NP];
    auto load_scales = [&](int b) {
        const uint8_t *base[NP];
        int64_t at[NP], total[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int idx = tid * NP + j, r = idx >> 1;
            const bool isb = r >= TM;
            const int64_t R = isb ? p.Rb : p.Ra, want = isb ? n0 + r - TM : m0 + r;
            base[j] = isb ? p.bs : p.as;
            at[j] = (want < R - 1 ? want : R - 1) * (int64_t)nkb + b * 32 + (idx & 1) * 16;
            total[j] = R * (int64_t)nkb;
        }
        if (b * 32 + 32 <= nkb) {  // (the same for all: both loads are out before anything waits)
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const Bytes16 t = *reinterpret_cast<const Bytes16 *>(base[j] + at[j]);
                piece[j] = make_uint4(t.v[0], t.v[1], t.v[2], t.v[3]);
            }
            return;
        }
        // The ragged end of a row, zeros behind it: 16 bytes from the row's place or from the end of the whole array,
        // whichever comes first, shifted and masked.  (A load per byte took 5 us of every 128 x 256 tile: 64 requests an
        // instruction.)
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int left = nkb - b * 32 - ((tid * NP + j) & 1) * 16;
            const int64_t from = at[j] < total[j] - 16 ? at[j] : total[j] - 16;
            uint64_t lo = 0, hi = 0;
            if (left > 0 && from >= 0) {
                const Bytes16 t = *reinterpret_cast<const Bytes16 *>(base[j] + from);
                const int sh = 8 * (int)(at[j] - from);  // 0 .. 120: at least one byte of the row is among the 16
                lo = t.v[0] | (uint64_t)t.v[1] << 32;
                hi = t.v[2] | (uint64_t)t.v[3] << 32;
                if (sh >= 64) {
                    lo = hi >> (sh - 64);
                    hi = 0;
                } else if (sh > 0) {
                    lo = lo >> sh | hi << (64 - sh);
                    hi >>= sh;
                }
                if (left < 8) lo &= (uint64_t(1) << (8 * left)) - 1;
                if (left <= 8) hi = 0;
                else if (left < 16) hi &= (uint64_t(1) << (8 * (left - 8))) - 1;
            } else if (left > 0) {  // an array of less than 16 bytes
                for (int k = 0; k < left; ++k) {
                    const uint64_t byte = base[j][at[j] + k];
                    if (k < 8) lo |= byte << (8 * k);
                    else hi |= byte << (8 * (k - 8));
                }
            }
            piece[j] = make_uint4((uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32));
        }
    };
    // 8-byte slot t (0..3) of a row sits at slot t ^ (row / 8 % 4): the fragment reads of 32 rows touch every bank once
    auto write_scales = [&]() {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int idx = tid * NP + j, r = idx >> 1, sw = (r >> 3) & 3, t = (idx & 1) * 2;
            if (ROWS * 2 % (64 * WAVES) != 0 && r >= ROWS) break;  // (128 x 64 tile: 192 rows on 256 threads)
            uint8_t *dst = smem + Tile::OFF_S + r * 32;
            *reinterpret_cast<uint2 *>(dst + ((t ^ sw) << 3)) = make_uint2(piece[j].x, piece[j].y);
            *reinterpret_cast<uint2 *>(dst + (((t + 1) ^ sw) << 3)) = make_uint2(piece[j].z, piece[j].w);
        }
    };

    // fragment reads
    const int fr = lane & 31, fh = lane >> 5;
    const int fm = (fr & 7) ^ ((fr >> 3) & 1);
    const uint32_t fl0 = (uint32_t)((fr >> 3) * 1024 + (fr & 7) * 128);
    uint32_t foff[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) foff[kk] = fl0 + (uint32_t)((((kk << 1) | fh) ^ fm) << 4);
    const uint32_t perm_sel = FMT ? (fh ? 0x03010301u : 0x02000200u) : (fh ? 0x07050301u : 0x06040200u);
    auto frag_scale = [&](int s, int row) {  // the lane's scale bytes of stage s, byte k = instruction K-step k
        const int slot = FMT ? (s & 7) >> 1 : s & 3;
        const uint8_t *q = smem + Tile::OFF_S + row * 32 + ((slot ^ ((row >> 3) & 3)) << 3);
        if (FMT) return (int)__builtin_amdgcn_perm(0u, *reinterpret_cast<const uint32_t *>(q + (s & 1) * 4), perm_sel);
        const uint2 w = *reinterpret_cast<const uint2 *>(q);
        return (int)__builtin_amdgcn_perm(w.y, w.x, perm_sel);
    };

    v16f acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // One phase multiplies one set of fragments while the next set is read.  E2M1: a stage is four phases of one K-step;
    // E4M3: two, of one K-step of two fragments.  The barrier stands before a stage's last phase: by then everyone holds
    // the stage's last fragments, so its buffer is free, and the reads of the next stage's first fragments and scale
    // bytes run under the last phase's matrix instructions.
    constexpr int PH = FMT ? 2 : 4, NF = FMT ? 2 : 1;
    v4i fa[2][WM][NF], fb[2][WN][NF];
    int sa[WM], sb[WN], sa_next[WM], sb_next[WN];
    int cur = 0;  // stage buffer of stage s
    auto read_frags = [&](int buf, int ph, int set) {
        const uint8_t *pa = smem + buf * Tile::STAGE + wm * WM * 4096;
        const uint8_t *pb = smem + buf * Tile::STAGE + TM * 128 + wn * WN * 4096;
#pragma unroll
        for (int h = 0; h < NF; ++h) {
#pragma unroll
            for (int j = 0; j < WN; ++j)
                fb[set][j][h] = *reinterpret_cast<const v4i *>(pb + j * 4096 + foff[ph * NF + h]);
#pragma unroll
            for (int i = 0; i < WM; ++i)
                fa[set][i][h] = *reinterpret_cast<const v4i *>(pa + i * 4096 + foff[ph * NF + h]);
        }
    };
    auto read_scales = [&](int s) {
#pragma unroll
        for (int i = 0; i < WM; ++i) sa_next[i] = frag_scale(s, wm * 32 * WM + 32 * i + fr);
#pragma unroll
        for (int j = 0; j < WN; ++j) sb_next[j] = frag_scale(s, TM + wn * 32 * WN + 32 * j + fr);
    };
    auto take_scales = [&]() {
#pragma unroll
        for (int i = 0; i < WM; ++i) sa[i] = sa_next[i];
#pragma unroll
        for (int j = 0; j < WN; ++j) sb[j] = sb_next[j];
    };
    auto multiply = [&](auto phase) {  // (the byte of the scale register is an instruction field)
        constexpr int ph = decltype(phase)::value, set = ph & 1;
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                const v4i b0 = fb[set][j][0], a0 = fa[set][i][0];
                v8i b8 = {b0.x, b0.y, b0.z, b0.w, 0, 0, 0, 0}, a8 = {a0.x, a0.y, a0.z, a0.w, 0, 0, 0, 0};
                if constexpr (FMT) {
                    const v4i b1 = fb[set][j][NF - 1], a1 = fa[set][i][NF - 1];
                    b8 = (v8i){b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
                    a8 = (v8i){a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                }
                acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b8, a8, acc[i][j], FMT ? 0 : 4, FMT ? 0 : 4,
                                                                            ph, sb[j], ph, sa[i]);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto all_but_last = [&]() {  // phases 0 .. PH-2 of the stage in buffer cur
        read_frags(cur, 1, 1);
        multiply(IC<0>{});
        if constexpr (PH == 4) {
            read_frags(cur, 2, 0);
            multiply(IC<1>{});
            read_frags(cur, 3, 1);
            multiply(IC<2>{});
        }
    };
    if (nstages > 0) {
        load_scales(0);
#pragma unroll
        for (int s = 0; s < NBUF; ++s)
            if (s < nstages) issue(s, s);
        write_scales();  // (the compiler waits for the bytes, and with them for all loads that are out)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (nbatches > 1) load_scales(1);
        read_frags(0, 0, 0);
        read_scales(0);
        take_scales();
        for (int s = 0; s + 1 < nstages; ++s) {
            all_but_last();
            // (a use of the sums: keeps the compiler from moving the matrix instructions behind the branches below)
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j) asm volatile("" : "+v"(acc[i][j]));
            // stage s+1 has landed (the loads of the stages after it may be out), everyone is done with buffer cur
            if (s + NBUF - 1 < nstages)
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NL * (NBUF - 2)) : "memory");
            else
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if ((s + 1) % BATCH == 0) {
                write_scales();
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if ((s + 1) / BATCH + 1 < nbatches) load_scales((s + 1) / BATCH + 1);
            }
            const int next = cur == NBUF - 1 ? 0 : cur + 1;
            read_frags(next, 0, 0);
            read_scales(s + 1);
            if (s + NBUF < nstages) issue(s + NBUF, cur);
            multiply(IC<PH - 1>{});
            take_scales();
            cur = next;
        }
        all_but_last();
        multiply(IC<PH - 1>{});
    }

    // epilogue: every wave transposes 32 rows at a time through its own slice of the stage buffers (row of 128 WN bytes,
    // 16-byte chunk c of row r at chunk c ^ r) and stores whole row pieces
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    constexpr int PITCH = 128 * WN, CHUNKS = 8 * WN;
    static_assert(WAVES * 32 * PITCH <= NBUF * Tile::STAGE, "32 rows of every wave must fit the stage buffers");
    uint8_t *epi = smem + wave * (32 * PITCH);
    constexpr int RPI = 64 / CHUNKS;  // rows per store instruction
    const int rl = lane / CHUNKS, ch = lane % CHUNKS;
    const int64_t col = n0 + wn * 32 * WN + ch * 4;
    const int64_t left = p.Rb - col;
    const bool whole = (p.vec & 1) && left >= 4;
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      // Values added to: all at once (rows beyond the last are the last again, for nobody), and all added before the first store, since a wait
      // for a load is one for the stores before it too.  us, one by one in front of their stores / loaded at once but added one by one / like
      // this: 6656 x 11008 x 768 198 / 148 / 146, 768 x 800 x 256 4.4 / 4.6 / 4.1, 3520 x 2304 x 896 20.1 / 20.9 / 19.4.
      // The wide tile, one per compute unit, loads them before its way through LDS (13888 x 6912 x 576 193, behind it 194; 6688 x 3072 x 992 46.6,
      // 47.4), the others, several there, behind it: beside a product that is not added to, M x N x K of the layer, 2400 x 256 x 4352 14.7, behind
      // it 14.1 (one by one 14.1), 2048 x 256 x 4864 13.3, 12.7 (12.6), 256 x 2048 x 1536 9.0, 8.8 (8.8).
      constexpr int NU = 32 / RPI;
      const int64_t row0 = m0 + wm * 32 * WM + 32 * i + rl;
      const bool add = ACC && p.accumulate && whole;
      v4f v[NU], old[NU];
      auto load_old = [&]() {
        if (!add) return;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int64_t row = row0 + u * RPI < p.Ra ? row0 + u * RPI : p.Ra - 1;
            old[u] = *reinterpret_cast<const v4f *>(reinterpret_cast<const float *>(p.out) + row * p.ld + col);
        }
      };
      if constexpr (WN > 1) load_old();
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int c = j * 8 + qd * 2 + fh;
            *reinterpret_cast<v4f *>(epi + fr * PITCH + ((c ^ (fr & (CHUNKS - 1))) << 4)) =
                (v4f){acc[i][j][4 * qd + 0], acc[i][j][4 * qd + 1], acc[i][j][4 * qd + 2], acc[i][j][4 * qd + 3]};
        }
      auto read = [&](int u) {
        const int r = u * RPI + rl;
        return *reinterpret_cast<const v4f *>(epi + r * PITCH + ((ch ^ (r & (CHUNKS - 1))) << 4));
      };
      if constexpr (WN == 1) load_old();
      if constexpr (ACC) {
#pragma unroll
        for (int u = 0; u < NU; ++u) v[u] = read(u);
        if (add) {
#pragma unroll
          for (int u = 0; u < NU; ++u) v[u] += old[u];
        }
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if constexpr (!ACC) v[u] = read(u);
        if (row0 + u * RPI < p.Ra) store4<ACC>(p, row0 + u * RPI, col, left, whole, v[u]);
      }
    }
}

// ---- ragged-shape kernel, 32 x 32 tiles: few outputs --------------------------------------------
// 24 x 6144 x 4096 makes 96 tiles of 64 x 64, and a tile of them is one serial chain: 730 clocks per stage of 128 bytes of K (8.0 us),
// most of it fragment reads waited for one K-step at a time, and two thirds of the chip idle.  Here a stage's chain is as short
// as could be made:
//   * four waves on a 32 x 32 tile, V_MFMA_SCALE_F32_16X16X128_F8F6F4, one accumulator each (17 clocks per instruction in a chain on one
//     accumulator, 24 to 33 where several alternate); the next stage's fragments are read under this one's instructions;
//   * one barrier per stage and no branch in it: a stage that does not exist is "loaded" with no lane active, so that the wait
//     counts stay constants; the ragged last stage is moved back to end with the row;
//   * a fifth wave brings the scale bytes (8-byte loads at any alignment, 64 bytes per row in a batch, written to LDS a batch ahead):
//     its waits hold up nobody's direct-to-LDS loads.
// NBUF stage buffers: 4 (40 KiB, four workgroups per compute unit) or 8 (72 KiB).  Rows are of at least 128 bytes of codes (small_gains), or empty.
// Measured back to back in a graph, bf16 output, 64 x 64 tiles / this: MXFP4 24 x 6144 x 4096 8.0 / 5.6 us, 256 x 512 x 512
// 4.1 / 3.6, 100 x 1000 x 14336 20.6 / 12.1, 500 x 1000 x 1440 6.3 / 5.5; MXFP8 24 x 6144 x 4096 11.1 / 7.2.  What is left at 24 x 6144
// x 4096: 1.7 us of launch, 1.4 us until the first stage and its scale bytes are there, 0.12 us per stage.
// The same on 64 x 64 tiles (V_MFMA_SCALE_F32_32X32X64_F8F6F4) was 20 % faster than gemm_edge_kernel's from 32 stages on and
// slower below 16: not built.
constexpr int SMALL = 32;                        // output tile edge
constexpr int SMALL_STAGE = 2 * SMALL * 128;     // bytes of codes per stage: A's 32 rows, then B's
constexpr int SMALL_SC = 2 * SMALL * 64;         // a batch of scale bytes

template <int FMT, int NBUF>
__global__ __launch_bounds__(320) void gemm_small_kernel(const EdgeGemm p0, const EdgeGemm p1, const uint32_t groups0)
{
    const bool second = blockIdx.x >= groups0;  // uniform
    const EdgeGemm &p = second ? p1 : p0;
    const uint32_t bid = blockIdx.x - (second ? groups0 : 0u);
    constexpr int T = SMALL, OFF_SB = NBUF * SMALL_STAGE;
    constexpr int SB = FMT ? 4 : 8;   // scale bytes per row and stage
    constexpr int BATCH_STAGES = 64 / SB;
    static_assert(scale_batch_drained(2, BATCH_STAGES) && scale_batch_in_time(1, BATCH_STAGES), "scale buffers refilled too early or too late");
    __shared__ __attribute__((aligned(1024))) uint8_t smem[OFF_SB + 2 * SMALL_SC];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int64_t m0, n0;
    if (!edge_has_tile(p, bid)) return;
    edge_tile(p, bid, T, T, m0, n0);
    const int rowbytes = (int)(FMT ? p.C : (p.C >> 1)), nkb = (int)(p.C >> 5);
    const int nstages = (rowbytes + 127) >> 7;

    if (wave == 4) {
        // ---- the wave that brings the scale bytes ----
        // piece j of a batch: a lane's 8 bytes (slot lane % 8 of the batch's 64) of row 8 j + lane / 8 (A's rows, then B's)
        constexpr int NP = 2 * T / 8;
        const int nbatches = (nkb + 63) >> 6;
        const int valid = nkb - SB * (nstages - 1);  // bytes of the last stage
        uint2 piece[NP];
        auto load = [&](int b) {
            const int col = b * 64 + (lane & 7) * 8;
            int last[2], lastrow[2];  // of A, of B
            const uint8_t *base[2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int64_t r0 = o ? n0 : m0, R = o ? p.Rb : p.Ra, room = (R - r0) * nkb;
                base[o] = (o ? p.bs : p.as) + r0 * nkb;
                lastrow[o] = (int)(R - r0 < T ? R - r0 : T) - 1;
                last[o] = (int)(room < (1 << 30) ? room : (1 << 30)) - 8;  // the last place that 8 bytes can be loaded from
            }
            auto place = [&](int j) {
                const int o = j >= NP / 2, want = (j % (NP / 2)) * 8 + (lane >> 3);
                return (want < lastrow[o] ? want : lastrow[o]) * nkb + (col < nkb ? col : 0);
            };
            if ((p.Ra < p.Rb ? p.Ra : p.Rb) * nkb >= 8) {
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const int o = j >= NP / 2, at = place(j);
                    const Bytes8 t = *reinterpret_cast<const Bytes8 *>(base[o] + (at < last[o] ? at : last[o]));
                    piece[j] = make_uint2(t.v[0], t.v[1]);
                }
                // (the last bytes of a whole array are loaded from further ahead)
                const int64_t end = (int64_t)(T - 1) * nkb + (nkb + 7) / 8 * 8;
                if (last[0] + 8 < end || last[1] + 8 < end) {
#pragma unroll
                    for (int j = 0; j < NP; ++j) {
                        const int o = j >= NP / 2, at = place(j);
                        const uint64_t v = (piece[j].x | (uint64_t)piece[j].y << 32) >> (at > last[o] ? 8 * (at - last[o]) : 0);
                        piece[j] = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
                    }
                }
            } else {  // an array of less than 8 bytes
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const int at = place(j);
                    uint64_t v = 0;
#pragma unroll 1
                    for (int k = 0; k < 8 && k < nkb - col; ++k) v |= (uint64_t)base[j >= NP / 2][at + k] << (8 * k);
                    piece[j] = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
                }
            }
        };
        auto write = [&](int b) {
            if (b == nbatches - 1 && valid < SB) {
                // the last stage's codes are moved back to end with the row: so are its scale bytes, zeros in front of them for the
                // blocks that the stage before has had (products below 2^-254 * 2^24)
                auto fix = [&](uint64_t v) { return v << (8 * (SB - valid)); };
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const int s = b * BATCH_STAGES + (lane & 7) * (FMT ? 2 : 1);
                    uint32_t x = piece[j].x, y = piece[j].y;
                    if (FMT) {
                        if (s == nstages - 1) x = (uint32_t)fix(x);
                        if (s + 1 == nstages - 1) y = (uint32_t)fix(y);
                    } else if (s == nstages - 1) {
                        const uint64_t v = fix(x | (uint64_t)y << 32);
                        x = (uint32_t)v, y = (uint32_t)(v >> 32);
                    }
                    piece[j] = make_uint2(x, y);
                }
            }
            // slot t of a row sits at slot t ^ (row % 16) / 4: the reads of 16 rows touch every bank once
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int r = j * 8 + (lane >> 3);
                *reinterpret_cast<uint2 *>(smem + OFF_SB + (b & 1) * SMALL_SC + r * 64 + (((lane & 7) ^ ((r & 15) >> 2)) << 3)) = piece[j];
            }
        };
        if (nstages == 0) return;
        load(0);
        write(0);
        if (nbatches > 1) load(1);
        for (int s = 0; s <= nstages; ++s) {  // (as many barriers as the others have)
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            // Batch b goes where batch b - 2 was: one stage after its last stage was read, since the others pass the barrier in between
            // with those reads on their way (its waits are for their loads) and have the bytes in registers at this one.
            const int b = s / BATCH_STAGES + 1;
            if (s == scale_batch_barrier(b, BATCH_STAGES) && b < nbatches) {
                write(b);
                if (b + 1 < nbatches) load(b + 1);
            }
        }
        return;
    }

    // ---- the four waves that multiply ----
    const int wm = wave >> 1, wn = wave & 1;
    // Direct-to-LDS loads: waves 0 and 1 bring A's rows, 2 and 3 B's, 16 rows each; load n of a wave moves 8 (its immediate offset,
    // which the instruction adds to both addresses, is taken off the lane's).  Chunk c of row r of 8-row group g sits at slot
    // c ^ r ^ 5 (g & 1) of the row, which spreads the 16-byte reads of 16 rows over all banks.
    const bool isb = wave >= 2;
    const int64_t r0 = isb ? n0 : m0, rows = (isb ? p.Rb : p.Ra) - r0;
    const int lastrow = (int)(rows < T ? rows : T) - 1;
    constexpr int BIAS = 1024;  // keeps the lanes' offsets from falling below 0
    const uint8_t *src = (isb ? p.bq : p.aq) + r0 * rowbytes - BIAS;
    uint32_t voff[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int want = (wave & 1) * 16 + n * 8 + (lane >> 3), chunk = ((lane & 7) ^ (lane >> 3) ^ n * 5) << 4;
        voff[n] = (uint32_t)((want < lastrow ? want : lastrow) * rowbytes + chunk + BIAS - n * 1024);
    }
    const uint32_t lds_dst = lds0 + (uint32_t)wave * 2048u;
    const int koff_last = rowbytes - 128;
    auto issue = [&](int s, uint32_t to) {  // stage s into buffer `to`
        const uint8_t *at = src + (s * 128 < koff_last ? s * 128 : koff_last);
        const int on = __builtin_amdgcn_readfirstlane(s < nstages ? -1 : 0);
        asm volatile("s_mov_b32 m0, %0\n\ts_mov_b32 exec_lo, %1\n\ts_mov_b32 exec_hi, %1\n\tglobal_load_lds_dwordx4 %2, %4\n\t"
                     "global_load_lds_dwordx4 %3, %4 offset:1024\n\ts_mov_b64 exec, -1" ::"s"(lds_dst + to * SMALL_STAGE), "s"(on),
                     "v"(voff[0]), "v"(voff[1]), "s"(at)
                     : "memory");
    };

    // fragments: a lane holds chunks kb and 4 + kb of row lane % 16's 128 bytes (E2M1: of the stage's two K-steps, E4M3: both halves
    // of its one)
    const int r16 = lane & 15, kb = lane >> 4, g1 = (lane >> 3) & 1, r7 = lane & 7;
    const uint32_t foff = (uint32_t)(g1 * 1024 + r7 * 128 + ((kb ^ r7 ^ g1 * 5) << 4));
    const uint8_t *fa_at[2], *fb_at[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        fa_at[h] = smem + (foff ^ (uint32_t)(h << 6)) + wm * 2048;
        fb_at[h] = smem + (foff ^ (uint32_t)(h << 6)) + T * 128 + wn * 2048;
    }
    const uint8_t *sa_at = smem + OFF_SB + (wm * 16 + r16) * 64, *sb_at = smem + OFF_SB + (T + wn * 16 + r16) * 64;
    // byte i of the register: the scale of block 4 i + kb of the stage
    const uint32_t perm_sel = FMT ? (uint32_t)kb : (uint32_t)(kb | (4 + kb) << 8);
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    v4i fa[2][2], fb[2][2];
    uint2 ra[2], rb[2];
    auto read_stage = [&](int s, int buf, auto set_) {
        constexpr int set = decltype(set_)::value;
        const int in = s & (BATCH_STAGES - 1), slot = FMT ? in >> 1 : in;
        const int at = ((s / BATCH_STAGES) & 1) * SMALL_SC + ((slot ^ (r16 >> 2)) << 3) + (FMT ? (in & 1) * 4 : 0);
        if (FMT) {
            ra[set] = make_uint2(*reinterpret_cast<const uint32_t *>(sa_at + at), 0u);
            rb[set] = make_uint2(*reinterpret_cast<const uint32_t *>(sb_at + at), 0u);
        } else {
            ra[set] = *reinterpret_cast<const uint2 *>(sa_at + at);
            rb[set] = *reinterpret_cast<const uint2 *>(sb_at + at);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            fb[set][h] = *reinterpret_cast<const v4i *>(fb_at[h] + buf * SMALL_STAGE);
            fa[set][h] = *reinterpret_cast<const v4i *>(fa_at[h] + buf * SMALL_STAGE);
        }
    };
    if (nstages > 0) {
#pragma unroll
        for (int s = 0; s < NBUF - 1; ++s) issue(s, s);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * (NBUF - 2)) : "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): with scalar loads still out the loop could not wait for single reads
        read_stage(0, 0, IC<0>{});
        int s = 0;
        // Stage s, buffer j, register set j % 2: stage s + 1 has landed, everyone has the fragments of stage s - 1.  (After the last
        // stage this reads a buffer that nothing was loaded into, for nobody.)
        auto advance = [&](auto j_) {
            constexpr int j = decltype(j_)::value, set = j & 1;
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * (NBUF - 3)) : "memory");
            const int sa = (int)__builtin_amdgcn_perm(ra[set].y, ra[set].x, perm_sel);
            const int sb = (int)__builtin_amdgcn_perm(rb[set].y, rb[set].x, perm_sel);
            read_stage(s + 1, (j + 1) % NBUF, IC<1 - set>{});
            issue(s + NBUF - 1, (j + NBUF - 1) % NBUF);
            const v4i b0 = fb[set][0], a0 = fa[set][0], b1 = fb[set][1], a1 = fa[set][1];
            if constexpr (FMT) {
                const v8i b8 = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w}, a8 = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b8, a8, acc, 0, 0, 0, sb, 0, sa);
            } else {
                const v8i b8 = {b0.x, b0.y, b0.z, b0.w, 0, 0, 0, 0}, a8 = {a0.x, a0.y, a0.z, a0.w, 0, 0, 0, 0};
                acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b8, a8, acc, 4, 4, 0, sb, 0, sa);
                const v8i b9 = {b1.x, b1.y, b1.z, b1.w, 0, 0, 0, 0}, a9 = {a1.x, a1.y, a1.z, a1.w, 0, 0, 0, 0};
                acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b9, a9, acc, 4, 4, 1, sb, 1, sa);
            }
            __builtin_amdgcn_sched_barrier(0);
            ++s;
        };
        for (;;) {
#define MXFP4_ADVANCE(J)                    \
    if constexpr ((J) < NBUF) {             \
        advance(IC<(J) < NBUF ? (J) : 0>{}); \
        if (s == nstages) goto done;        \
    }
            MXFP4_ADVANCE(0) MXFP4_ADVANCE(1) MXFP4_ADVANCE(2) MXFP4_ADVANCE(3)
            MXFP4_ADVANCE(4) MXFP4_ADVANCE(5) MXFP4_ADVANCE(6) MXFP4_ADVANCE(7)
#undef MXFP4_ADVANCE
        }
    }
done:
    // a lane holds columns 4 kb .. +3 of row r16 of the wave's 16 x 16: straight to memory
    const int64_t row = m0 + wm * 16 + r16, col = n0 + wn * 16 + 4 * kb;
    const int64_t left = p.Rb - col;
    if (row >= p.Ra) return;
    const bool whole = (p.vec & 1) && left >= 4;
    if (p.accumulate && whole) acc += *reinterpret_cast<const v4f *>(reinterpret_cast<const float *>(p.out) + row * p.ld + col);
    store4<true>(p, row, col, left, whole, acc);
}

// ---- ragged-shape kernel, 128 x 64 tiles, rows of at most two stages ------------------------------
// 256 bytes of codes per row are 16 matrix instructions per wave and tile: what such a product takes is the writing of its output,
// and on gemm_edge_kernel's tiles, of which a compute unit holds one or two, it took 2 to 2.5 times as long as that (a tile's first loads, its
// few instructions and its stores one after the other, the rows of a bf16 tile stored in 64-byte pieces).  Here a workgroup loads its whole
// contraction at once and keeps no ring: S stages of 24 KiB and 3 KiB of scale bytes, five or three workgroups per compute unit, whose
// loads, instructions and stores overlap; the output leaves in 128- or 256-byte rows of the tile, past the caches where these are whole
// lines, else through them, so that neighbouring tiles' halves of a line meet.
// Measured back to back in a graph, us, gemm_edge_kernel on the tiles it was given / this: MXFP4, bf16 output, 9624 x 20560 x 32 218 / 99 (4.0
// TB/s of output), 12008 x 3400 x 512 43.1 / 32.0, 12526 x 9728 x 256 80 / 55, 2273 x 7832 x 256 19.6 / 12.1, rows of 3003 elements 2000 x 3000 x 480
// 13.2 / 9.7; fp32 8192 x 8192 x 512 69.9 / 62.6, added to 2048 x 3072 x 384 13.7 / 10.8; MXFP8 12008 x 3400 x 256 41.2 / 30.4.  With three
// stages (75 KiB, two workgroups per unit) it was the slower: 2048 x 3072 x 768 9.2 / 9.9.
template <int S>
struct ShortTile {
    static constexpr int TM = 128, TN = 64, ROWS = TM + TN, STAGE = ROWS * 128, OFF_S = S * STAGE, LDS = OFF_S + ROWS * 16;
};

template <int FMT, int S>
__global__ __launch_bounds__(256) void gemm_short_kernel(const EdgeGemm p0, const EdgeGemm p1, const uint32_t groups0)
{
    const bool second = blockIdx.x >= groups0;  // uniform
    const EdgeGemm &p = second ? p1 : p0;
    const uint32_t bid = blockIdx.x - (second ? groups0 : 0u);
    using Tile = ShortTile<S>;
    constexpr int TM = Tile::TM, TN = Tile::TN;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[Tile::LDS];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    int64_t m0, n0;
    if (!edge_has_tile(p, bid)) return;
    edge_tile(p, bid, TM, TN, m0, n0);
    const int rowbytes = (int)(FMT ? p.C : (p.C >> 1)), nkb = (int)(p.C >> 5);  // at most 128 S, 4 S (E4M3) or 8 S
    const int nstages = (rowbytes + 127) >> 7;
    const int last_a = (int)(p.Ra - m0 < TM ? p.Ra - m0 : TM) - 1, last_b = (int)(p.Rb - n0 < TN ? p.Rb - n0 : TN) - 1;

    // Scale bytes: 16 per row in LDS, zeros behind the end of the row (as in gemm_edge_kernel); piece i: 8 of them, of row (tid + 256 i) / 2
    uint64_t piece[2] = {0, 0};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int idx = tid + 256 * i, r = idx >> 1, col = (idx & 1) * 8, left = nkb - col;
        if (r >= Tile::ROWS || left <= 0) continue;
        const bool isb = r >= TM;
        const int64_t r0 = isb ? n0 : m0, total = (isb ? p.Rb : p.Ra) * nkb;
        const int want = isb ? r - TM : r, last = isb ? last_b : last_a;
        const int64_t at = (r0 + (want < last ? want : last)) * nkb + col;
        const uint8_t *base = isb ? p.bs : p.as;
        if (total >= 8) {
            const int64_t from = at < total - 8 ? at : total - 8;  // (the array's last bytes: loaded from further ahead)
            const Bytes8 t = *reinterpret_cast<const Bytes8 *>(base + from);
            piece[i] = (t.v[0] | (uint64_t)t.v[1] << 32) >> (8 * (int)(at - from));
        } else {
            for (int k = 0; k < left; ++k) piece[i] |= (uint64_t)base[at + k] << (8 * k);
        }
        if (left < 8) piece[i] &= (uint64_t(1) << (8 * left)) - 1;
    }
    // codes: load n of wave w and stage s moves 8-row group 6 w + n, chunks beyond the end of a row are its last one again
#pragma unroll
    for (int n = 0; n < 6; ++n) {
        const int group = wave * 6 + n;
        const bool isb = group >= TM / 8;
        const int want = (isb ? group - TM / 8 : group) * 8 + (lane >> 3), last = isb ? last_b : last_a;
        const uint8_t *base = isb ? p.bq + n0 * rowbytes : p.aq + m0 * rowbytes;
        const int row = (want < last ? want : last) * rowbytes, chunk = ((lane & 7) ^ (lane >> 3) ^ (n & 1)) << 4;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int at = s * 128 + chunk < rowbytes - 16 ? s * 128 + chunk : rowbytes - 16;
            if (s < nstages) dma16(lds0 + (uint32_t)(s * Tile::STAGE + group * 1024), (uint32_t)(row + at), base);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if (tid + 256 * i < 2 * Tile::ROWS)
            *reinterpret_cast<uint2 *>(smem + Tile::OFF_S + (tid + 256 * i) * 8) = make_uint2((uint32_t)piece[i], (uint32_t)(piece[i] >> 32));
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // fragments and scale bytes as in gemm_edge_kernel
    const int fr = lane & 31, fh = lane >> 5;
    const uint32_t foff = (uint32_t)((fr >> 3) * 1024 + (fr & 7) * 128 + ((fh ^ (fr & 7) ^ ((fr >> 3) & 1)) << 4));
    const uint32_t perm_sel = FMT ? (fh ? 0x03010301u : 0x02000200u) : (fh ? 0x07050301u : 0x06040200u);
    v16f acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        if (s >= nstages) break;
        const uint8_t *st = smem + s * Tile::STAGE;
        auto frag = [&](int row0, int kk) { return *reinterpret_cast<const v4i *>(st + row0 * 128 + (foff ^ (uint32_t)(kk << 5))); };
        auto scale = [&](int row0) {
            const uint8_t *q = smem + Tile::OFF_S + (row0 + fr) * 16 + s * (FMT ? 4 : 8);
            if (FMT) return (int)__builtin_amdgcn_perm(0u, *reinterpret_cast<const uint32_t *>(q), perm_sel);
            const uint2 w = *reinterpret_cast<const uint2 *>(q);
            return (int)__builtin_amdgcn_perm(w.y, w.x, perm_sel);
        };
        v4i fa[2][4], fb[4];
        int sa[2];
        const int sb = scale(TM + wn * 32);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) fb[kk] = frag(TM + wn * 32, kk);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            sa[i] = scale(wm * 64 + i * 32);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) fa[i][kk] = frag(wm * 64 + i * 32, kk);
        }
        auto step = [&](auto k_) {
            constexpr int k = decltype(k_)::value;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if constexpr (FMT) {
                    const v4i b0 = fb[2 * k], b1 = fb[2 * k + 1], a0 = fa[i][2 * k], a1 = fa[i][2 * k + 1];
                    const v8i b8 = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w}, a8 = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                    acc[i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b8, a8, acc[i], 0, 0, k, sb, k, sa[i]);
                } else {
                    const v4i b0 = fb[k], a0 = fa[i][k];
                    const v8i b8 = {b0.x, b0.y, b0.z, b0.w, 0, 0, 0, 0}, a8 = {a0.x, a0.y, a0.z, a0.w, 0, 0, 0, 0};
                    acc[i] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b8, a8, acc[i], 4, 4, k, sb, k, sa[i]);
                }
            }
        };
        step(IC<0>{}), step(IC<1>{});
        if constexpr (!FMT) step(IC<2>{}), step(IC<3>{});
    }

    // The tile is put together in LDS, 16-byte chunk c of row r at chunk c ^ r (mod the chunks of a row), and leaves in whole rows.
    const bool lines = p.vec & 4;
    if (!p.out_fp32) {
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // everyone has multiplied
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const int r = wm * 64 + i * 32 + fr, c = wn * 4 + qd;
                *reinterpret_cast<uint2 *>(smem + r * 128 + ((c ^ (r & 7)) << 4) + fh * 8) =
                    make_uint2(pack_bf16(acc[i][4 * qd], acc[i][4 * qd + 1]), pack_bf16(acc[i][4 * qd + 2], acc[i][4 * qd + 3]));
            }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        uint16_t *const out = reinterpret_cast<uint16_t *>(p.out) + m0 * p.ld + n0;
        const int cols = (int)(p.Rb - n0 < TN ? p.Rb - n0 : TN);
        if (p.vec & 2) {
            const int c = lane & 7;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int r = wave * 32 + it * 8 + (lane >> 3);
                const v4u v = *reinterpret_cast<const v4u *>(smem + r * 128 + ((c ^ (r & 7)) << 4));
                if (r > last_a) continue;
                uint16_t *o = out + r * p.ld + c * 8;
                if (c * 8 + 8 <= cols) {
                    if (lines) __builtin_nontemporal_store(v, reinterpret_cast<v4u *>(o));
                    else *reinterpret_cast<v4u *>(o) = v;
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (c * 8 + e < cols) o[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
                }
            }
        } else if (p.vec & 8) {  // rows of whole 4 bytes: two columns a lane
            const int c = lane & 31;
#pragma unroll 4
            for (int it = 0; it < 16; ++it) {
                const int r = wave * 32 + it * 2 + (lane >> 5);
                const uint32_t v = *reinterpret_cast<const uint32_t *>(smem + r * 128 + (((c >> 2) ^ (r & 7)) << 4) + (c & 3) * 4);
                if (r > last_a || c * 2 >= cols) continue;
                uint16_t *o = out + r * p.ld + c * 2;
                if (c * 2 + 1 < cols) *reinterpret_cast<uint32_t *>(o) = v;
                else *o = (uint16_t)v;
            }
        } else {
#pragma unroll 4
            for (int it = 0; it < 32; ++it) {
                const int r = wave * 32 + it;
                const uint16_t v = *reinterpret_cast<const uint16_t *>(smem + r * 128 + (((lane >> 3) ^ (r & 7)) << 4) + (lane & 7) * 2);
                if (r <= last_a && lane < cols) out[r * p.ld + lane] = v;
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {  // rows 32 i .. +31 of either half of the tile
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int r = wm * 32 + fr, c = wn * 8 + qd * 2 + fh;
            *reinterpret_cast<v4f *>(smem + r * 256 + ((c ^ (r & 15)) << 4)) =
                (v4f){acc[i][4 * qd], acc[i][4 * qd + 1], acc[i][4 * qd + 2], acc[i][4 * qd + 3]};
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        float *const out = reinterpret_cast<float *>(p.out) + m0 * p.ld + n0;
        const int cols = (int)(p.Rb - n0 < TN ? p.Rb - n0 : TN);
        auto tile_row = [&](int r) { return (r >> 5) * 64 + i * 32 + (r & 31); };
        if (p.vec & 1) {
            const int c = lane & 15;
            const bool whole = c * 4 + 4 <= cols, add = p.accumulate && whole;
            v4f v[4], old[4];  // (what they are added to: all loads and sums before the first store)
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int r = wave * 16 + it * 4 + (lane >> 4), row = tile_row(r);
                v[it] = *reinterpret_cast<const v4f *>(smem + r * 256 + ((c ^ (r & 15)) << 4));
                if (add) old[it] = *reinterpret_cast<const v4f *>(out + (row < last_a ? row : last_a) * p.ld + c * 4);
            }
            if (add) {
#pragma unroll
                for (int it = 0; it < 4; ++it) v[it] += old[it];
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int r = wave * 16 + it * 4 + (lane >> 4), row = tile_row(r);
                if (row > last_a) continue;
                float *o = out + row * p.ld + c * 4;
                if (whole) {
                    if (lines) __builtin_nontemporal_store(v[it], reinterpret_cast<v4f *>(o));
                    else *reinterpret_cast<v4f *>(o) = v[it];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c * 4 + e < cols) o[e] = p.accumulate ? (o[e] + v[it][e]) : v[it][e];
                }
            }
        } else {  // a column a lane
#pragma unroll 4
            for (int it = 0; it < 16; ++it) {
                const int r = wave * 16 + it, row = tile_row(r);
                const float v = *reinterpret_cast<const float *>(smem + r * 256 + (((lane >> 2) ^ (r & 15)) << 4) + (lane & 3) * 4);
                if (row > last_a || lane >= cols) continue;
                float *o = out + row * p.ld + lane;
                *o = p.accumulate ? *o + v : v;
            }
        }
    }
}

}  // namespace

// Compute units of the current device (MI355X: 256); asked once per process and device.
static int device_cus()
{
    static int cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return NUM_CUS;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = NUM_CUS;
        cached[dev] = n;
    }
    return cached[dev];
}

// the tiled kernel wants whole 256 x 256 tiles, K in whole stages (128 bytes of codes per row: 256 E2M1
// or 128 E4M3 elements) and at least 1024 (scale bytes are fetched 32 per row), and 16-byte aligned
// code rows and output rows
// (tile_n: 256, or 128 for the narrow tile, which exists for E2M1 operands only)
static bool tile_eligible(const GemmArgs &g, int tile_n = TILE)
{
    if (g.a_fmt != g.b_fmt) return false;  // mixed formats: any-shape kernel
    if (tile_n != TILE && g.a_fmt != 0) return false;
    const bool k_ok = g.C >= 1024 && (g.C % (g.a_fmt ? 128 : 256)) == 0;
    return k_ok && (g.Ra % TILE) == 0 && (g.Rb % tile_n) == 0 && (g.ld % 8) == 0 &&
           (reinterpret_cast<uintptr_t>(g.as) % 16) == 0 && (reinterpret_cast<uintptr_t>(g.bs) % 16) == 0 &&
           (g.Ra / TILE) * (g.Rb / TILE) < (1 << 30) && g.C < (int64_t(1) << 26);  // (64 code rows: 32-bit lane offsets)
}

static TileGemm tile_args(const GemmArgs &g, int tile_n = TILE)
{
    return TileGemm{g.aq, g.as, g.bq, g.bs, g.C, g.out, g.ld, (int)(g.Ra / TILE), (int)(g.Rb / tile_n)};
}

template <int AF, int BF>
static hipError_t launch_any_f(const GemmArgs &g, hipStream_t st)
{
    dim3 grid((unsigned)((g.Ra + 63) / 64), (unsigned)((g.Rb + 63) / 64));
    if (g.out_fp32) {
        if (g.accumulate)
            hipLaunchKernelGGL((gemm_any_kernel<true, true, AF, BF>), grid, dim3(256), 0, st, g.aq, g.as, g.bq, g.bs,
                               g.Ra, g.Rb, g.C, g.out, g.ld);
        else
            hipLaunchKernelGGL((gemm_any_kernel<true, false, AF, BF>), grid, dim3(256), 0, st, g.aq, g.as, g.bq, g.bs,
                               g.Ra, g.Rb, g.C, g.out, g.ld);
    } else {
        hipLaunchKernelGGL((gemm_any_kernel<false, false, AF, BF>), grid, dim3(256), 0, st, g.aq, g.as, g.bq, g.bs,
                           g.Ra, g.Rb, g.C, g.out, g.ld);
    }
    return hipGetLastError();
}

static EdgeGemm edge_args(const GemmArgs &g, int tm, int tn)
{
    const int64_t pitch = g.ld * (g.out_fp32 ? 4 : 2);
    auto rows_at = [&](int bytes) { return pitch % bytes == 0 && reinterpret_cast<uintptr_t>(g.out) % bytes == 0; };
    const int vec = rows_at(g.out_fp32 ? 16 : 8) + 2 * rows_at(16) + 4 * rows_at(128) + 8 * (rows_at(4) && !rows_at(16));
    return EdgeGemm{g.aq, g.as, g.bq, g.bs, g.Ra, g.Rb, g.C, g.out, g.ld, (int)((g.Ra + tm - 1) / tm), (int)((g.Rb + tn - 1) / tn),
                    g.out_fp32, g.accumulate, vec};
}
static uint32_t edge_groups(const EdgeGemm &p) { return ((uint32_t)(p.tiles_m * p.tiles_n) + 7u) & ~7u; }

template <int FMT, int WM, int WN, int NWN, int NBUF>
static hipError_t launch_edge_f(const GemmArgs &g0, const GemmArgs *g1, hipStream_t st)
{
    using Tile = EdgeTile<WM, WN, NWN, NBUF>;
    const EdgeGemm p0 = edge_args(g0, Tile::TM, Tile::TN), p1 = edge_args(g1 ? *g1 : g0, Tile::TM, Tile::TN);
    const uint32_t n0 = edge_groups(p0), n1 = g1 ? edge_groups(p1) : 0u;
    if (g0.accumulate || (g1 && g1->accumulate))
        hipLaunchKernelGGL((gemm_edge_kernel<FMT, WM, WN, NWN, NBUF, true>), dim3(n0 + n1), dim3(64 * Tile::WAVES), 0, st, p0, p1, n0);
    else
        hipLaunchKernelGGL((gemm_edge_kernel<FMT, WM, WN, NWN, NBUF, false>), dim3(n0 + n1), dim3(64 * Tile::WAVES), 0, st, p0, p1, n0);
    return hipGetLastError();
}

template <int FMT, int NBUF>
static hipError_t launch_small_f(const GemmArgs &g0, const GemmArgs *g1, hipStream_t st)
{
    const EdgeGemm p0 = edge_args(g0, SMALL, SMALL), p1 = edge_args(g1 ? *g1 : g0, SMALL, SMALL);
    const uint32_t n0 = edge_groups(p0), n1 = g1 ? edge_groups(p1) : 0u;
    hipLaunchKernelGGL((gemm_small_kernel<FMT, NBUF>), dim3(n0 + n1), dim3(320), 0, st, p0, p1, n0);
    return hipGetLastError();
}

// Estimated microseconds of gemm_edge_kernel on tm x tn tiles: rounds of the tiles that the chip holds at once, each
// `full` per kilobyte of code row (half of that where at most one of two workgroups per CU is there) plus what filling
// and emptying the pipeline costs.  They only rank the three tile shapes and this kernel among the others: the constants of
// the two small tiles are older than its third stage buffer, and over 548 sizes (256 to 16384 rows and columns, C = 1024 to
// 14336) the estimates are 1.16, 1.11 and 1.10 times the measured time of 64 x 64, 128 x 64 and 128 x 256 tiles on average
// (four in five between 0.86 and 1.44; 0.1 to 0.2 less where rows are not whole cache lines apart).  Where they matter: few
// tiles (200 x 4096 x 4096: 64 x 64 8.5, 128 x 64 10.1, 128 x 256 18.6 us), a round just overfull (2080 x 4320 x 1440: 27.6,
// 21.2, 23.2 us), many tiles (8192 x 6112 x 4064: 290, 254, 179 us).
static double edge_cost(const GemmArgs &g0, const GemmArgs *g1, int tm, int tn, int slots, double full, double fixed)
{
    auto tiles = [&](const GemmArgs &g) { return ((g.Ra + tm - 1) / tm) * ((g.Rb + tn - 1) / tn); };
    auto kbytes = [](const GemmArgs &g) { return (double)(g.a_fmt ? g.C : g.C / 2) / 1000.0; };
    const int64_t t0 = tiles(g0), t1 = g1 ? tiles(*g1) : 0, t = t0 + t1, left = t % slots;
    const double kb = ((double)t0 * kbytes(g0) + (g1 ? (double)t1 * kbytes(*g1) : 0.0)) / (double)t;
    double us = (double)(t / slots) * (full * kb + fixed);
    if (left) us += (slots > NUM_CUS && left <= NUM_CUS ? 0.5 : 1.0) * full * kb + fixed;
    return us;
}

// What gemm_edge_kernel takes: both operands of one format, lane offsets of 255 rows in 32 bits.
static bool edge_eligible(const GemmArgs &g)
{
    return g.a_fmt == g.b_fmt && g.C < (int64_t(1) << 24) && g.Ra < (int64_t(1) << 31);
}

static EdgeProduct edge_product(const GemmArgs &g)
{
    return EdgeProduct{g.Ra, g.Rb, g.a_fmt ? g.C : g.C / 2, g.ld * (g.out_fp32 ? 4 : 2), g.a_fmt != 0, g.out_fp32 != 0, g.accumulate != 0};
}
static bool runs_short(const GemmArgs &g0, const GemmArgs *g1)
{
    const EdgeProduct p0 = edge_product(g0), p1 = g1 ? edge_product(*g1) : p0;
    return runs_short(p0, g1 ? &p1 : nullptr);
}

// The tile shape with the lowest estimate for one product, or two of one format side by side, among those whose tiles, a
// workgroup each, make a grid that can be launched (us = NO_ROUTE: none does).
constexpr double NO_ROUTE = 1e30;

struct EdgeChoice {
    int tile;  // 0: 64 x 64, 1: 128 x 64, 2: 128 x 256
    double us;
};
static EdgeChoice choose_edge(const GemmArgs &g0, const GemmArgs *g1 = nullptr)
{
    auto cost = [&](int tm, int tn, int threads, int slots, double full, double fixed) {
        auto groups = [&](const GemmArgs &g) { return ((g.Ra + tm - 1) / tm * ((g.Rb + tn - 1) / tn) + 7) & ~int64_t(7); };
        if (!grid_fits(groups(g0) + (g1 ? groups(*g1) : 0), threads)) return NO_ROUTE;
        return edge_cost(g0, g1, tm, tn, slots, full, fixed);
    };
    EdgeChoice best{0, cost(64, 64, 256, 512, 6.4, 1.5)};
    // Short rows are bound by the stores at a tile's end, which the estimates do not tell apart: while the chip holds all the
    // 64 x 64 tiles at once, they are done first.  128 x 64 over 64 x 64, 257 to 512 tiles, up to 512 bytes of codes per row:
    // 0.96 to 1.22, 1.06 on average, and where the output is added to 1.04 to 1.50, 1.28 (10736 x 88 x 384, rows of 91
    // elements: 12.3 us, 8.6).
    auto tiles = [](const GemmArgs &g) { return (g.Ra + 63) / 64 * ((g.Rb + 63) / 64); };
    auto short_rows = [](const GemmArgs &g) { return (g.a_fmt ? g.C : g.C / 2) <= 512; };
    if (short_rows(g0) && (!g1 || short_rows(*g1)) && tiles(g0) + (g1 ? tiles(*g1) : 0) <= 2 * NUM_CUS) return best;
    // In a pair, an output that is added to behind at most two stages (the weight gradient of a few tokens) is all reading and writing, which the
    // wide tile, one per compute unit, does not overlap: M x N x K of the layer, 256 x 8192 x 2304 44.4 us, 128 x 64 tiles 33.7, 64 x 15424 x 1408
    // 82.8, 48.7; 104 layers of up to 512 tokens 0.84 times the time.
    const bool add_short = g1 && g1->accumulate && edge_stages(edge_product(*g1)) <= 2;
    const double mid = cost(128, 64, 256, 512, 9.3, 1.5), large = add_short ? NO_ROUTE : cost(128, 256, 512, 256, 10.5, 3.5);
    if (runs_short(g0, g1) && mid < NO_ROUTE) return EdgeChoice{1, mid};
    if (mid <= best.us) best = EdgeChoice{1, mid};
    if (large <= best.us) best = EdgeChoice{2, large};
    return best;
}

// Short products that one workgroup per CU covers stay on the any-shape kernel where its launch, 1 us shorter (no LDS, no
// stages), outweighs its stores of 2 or 4 bytes and its loads in the open: less than two whole stages (256 bytes) of codes
// per row, in MXFP8 less than three where the output has at most 16 rows or columns, and
//   * at most 16 columns (also with a workgroup on every other CU more), or without accumulation at most 32 rows or columns:
//     any-shape time over ragged-shape time 0.60 to 1.11, 0.78 on average;
//   * rows of the output that the ragged-shape kernel cannot store 4 elements at a time either, except one whole stage (up
//     to 64 bytes also with a workgroup on every other CU more): 0.70 to 1.19, 0.88;
//   * at most 64 bytes, columns in no whole 16s, no accumulation, half the CUs: 0.77 to 1.08, 0.91.
// Elsewhere 0.79 to 5, 1.36.  Measured back to back in a graph over 2400 sizes up to 20000 x 20000 x 2048: 16 x 16 x 32 2.0 us
// against 3.1, 1000 x 1000 x 128 with 1003 elements per row 4.0 against 4.4.  Both kernels give the same bits.
static bool short_product(const GemmArgs &g)
{
    const int64_t bytes = g.a_fmt ? g.C : g.C / 2, tiles = (g.Ra + 63) / 64 * ((g.Rb + 63) / 64);
    if (bytes >= (g.a_fmt && (g.Ra <= 16 || g.Rb <= 16) ? 384 : 256)) return false;
    if (g.Rb <= 16) return tiles <= NUM_CUS * 3 / 2;
    if (tiles <= NUM_CUS && !g.accumulate && (g.Ra <= 32 || g.Rb <= 32)) return true;
    if (g.ld % 4 != 0) return tiles <= NUM_CUS ? bytes != 128 : bytes <= 64 && tiles <= NUM_CUS * 3 / 2;
    return bytes <= 64 && g.Rb % 16 != 0 && !g.accumulate && tiles <= NUM_CUS / 2;
}

// A block that is not for the tiled kernels: the ragged-shape kernel or, where that cannot or is slower, the any-shape one.
static GemmRoute any_route(const GemmArgs &g)
{
    if (!edge_eligible(g)) return GemmRoute{ROUTE_ANY_SHAPE, NO_ROUTE};
    const EdgeChoice edge = choose_edge(g);
    if (short_product(g)) return GemmRoute{ROUTE_ANY_SHAPE, edge.us};  // (an estimate is needed beside another product only)
    return edge.us < NO_ROUTE ? GemmRoute{ROUTE_EDGE_64 + edge.tile, edge.us} : GemmRoute{ROUTE_ANY_SHAPE, NO_ROUTE};
}

template <int FMT, int S>
static hipError_t launch_short_f(const GemmArgs &g0, const GemmArgs *g1, hipStream_t st)
{
    using Tile = ShortTile<S>;
    const EdgeGemm p0 = edge_args(g0, Tile::TM, Tile::TN), p1 = edge_args(g1 ? *g1 : g0, Tile::TM, Tile::TN);
    const uint32_t n0 = edge_groups(p0), n1 = g1 ? edge_groups(p1) : 0u;
    hipLaunchKernelGGL((gemm_short_kernel<FMT, S>), dim3(n0 + n1), dim3(256), 0, st, p0, p1, n0);
    return hipGetLastError();
}

static hipError_t launch_edge(const GemmArgs &g0, const GemmArgs *g1, int tile, hipStream_t st)
{
    if (tile == 2) return g0.a_fmt ? launch_edge_f<1, 2, 2, 4, 3>(g0, g1, st) : launch_edge_f<0, 2, 2, 4, 3>(g0, g1, st);
    const EdgeProduct p0 = edge_product(g0), p1 = g1 ? edge_product(*g1) : p0;
    if (tile == 1 && runs_short(g0, g1)) {
        if (edge_stages(p0) <= 1 && edge_stages(p1) <= 1) return g0.a_fmt ? launch_short_f<1, 1>(g0, g1, st) : launch_short_f<0, 1>(g0, g1, st);
        return g0.a_fmt ? launch_short_f<1, 2>(g0, g1, st) : launch_short_f<0, 2>(g0, g1, st);
    }
    if (tile == 1) return g0.a_fmt ? launch_edge_f<1, 2, 1, 2, 3>(g0, g1, st) : launch_edge_f<0, 2, 1, 2, 3>(g0, g1, st);
    if (const int small = small_tiles(p0, g1 ? &p1 : nullptr)) {
        // (eight stage buffers with a workgroup per compute unit at most: 1.2 times as fast from 32 stages of operands that come
        // from memory on, the same or 0.97 times up to 16)
        const GemmArgs &longer = g1 && g1->C > g0.C ? *g1 : g0;
        if (small <= NUM_CUS && (longer.a_fmt ? longer.C : longer.C / 2) > 16 * 128)
            return g0.a_fmt ? launch_small_f<1, 8>(g0, g1, st) : launch_small_f<0, 8>(g0, g1, st);
        return g0.a_fmt ? launch_small_f<1, 4>(g0, g1, st) : launch_small_f<0, 4>(g0, g1, st);
    }
    return g0.a_fmt ? launch_edge_f<1, 1, 1, 2, 4>(g0, g1, st) : launch_edge_f<0, 1, 1, 2, 4>(g0, g1, st);
}

static hipError_t launch_any(const GemmArgs &g, hipStream_t st)
{
    const GemmRoute r = any_route(g);
    if (r.kind != ROUTE_ANY_SHAPE) return launch_edge(g, nullptr, r.kind - ROUTE_EDGE_64, st);
    if (g.a_fmt == 0) return g.b_fmt == 0 ? launch_any_f<0, 0>(g, st) : launch_any_f<0, 1>(g, st);
    return g.b_fmt == 0 ? launch_any_f<1, 0>(g, st) : launch_any_f<1, 1>(g, st);
}

// rows r0.. (n of them) of A and columns c0.. (m of them) of B: the same problem on a sub-block of the output
static GemmArgs sub_block(const GemmArgs &g, int64_t r0, int64_t n, int64_t c0, int64_t m)
{
    GemmArgs h = g;
    const int64_t nkb = g.C / 32;
    h.aq = g.aq + r0 * (g.a_fmt ? g.C : g.C / 2);
    h.as = g.as + r0 * nkb;
    h.bq = g.bq + c0 * (g.b_fmt ? g.C : g.C / 2);
    h.bs = g.bs + c0 * nkb;
    h.Ra = n;
    h.Rb = m;
    h.out = static_cast<uint8_t *>(g.out) + (r0 * g.ld + c0) * (g.out_fp32 ? 4 : 2);
    return h;
}

template <int FMT, int NJ>
static hipError_t launch_tiled_f(const GemmArgs &g, hipStream_t st)
{
    const TileGemm p = tile_args(g, 64 * NJ);
    // persistent: one workgroup per CU (the kernel takes all of a CU's LDS) walks several tiles
    const int T = p.tiles_m * p.tiles_n;
    const int cus = device_cus();
    dim3 grid((unsigned)(T < cus ? T : cus));
    if (g.out_fp32) {
        if (g.accumulate)
            hipLaunchKernelGGL((gemm_tile_kernel<true, true, FMT, NJ>), grid, dim3(256), 0, st, p);
        else
            hipLaunchKernelGGL((gemm_tile_kernel<true, false, FMT, NJ>), grid, dim3(256), 0, st, p);
    } else {
        hipLaunchKernelGGL((gemm_tile_kernel<false, false, FMT, NJ>), grid, dim3(256), 0, st, p);
    }
    return hipGetLastError();
}

// whole rounds on 256 x 256 tiles, then the last round's tiles in halves (see gemm_tile_tail_kernel)
static hipError_t launch_tiled_tail(const GemmArgs &g, int64_t main_tiles, hipStream_t st)
{
    const TileGemm p = tile_args(g);
    dim3 grid((unsigned)device_cus());
    if (g.out_fp32) {
        if (g.accumulate)
            hipLaunchKernelGGL((gemm_tile_tail_kernel<true, true>), grid, dim3(256), 0, st, p, (int)main_tiles);
        else
            hipLaunchKernelGGL((gemm_tile_tail_kernel<true, false>), grid, dim3(256), 0, st, p, (int)main_tiles);
    } else {
        hipLaunchKernelGGL((gemm_tile_tail_kernel<false, false>), grid, dim3(256), 0, st, p, (int)main_tiles);
    }
    return hipGetLastError();
}

// whole 256 x 256 tiles not asked for: see RAG at gemm_tile_body (128 output rows of ld elements in 31-bit offsets)
static bool rag_eligible(const GemmArgs &g)
{
    return g.a_fmt == g.b_fmt && g.C >= 1024 && g.C < (int64_t(1) << 24) && g.Ra >= TILE && g.Rb >= TILE &&
           (g.Rb % 8) == 0 && (g.ld % 8) == 0 && g.ld < (1 << 21) && ((g.Ra + TILE - 1) / TILE) * ((g.Rb + TILE - 1) / TILE) < (1 << 29);
}

// tiles of 256 x 256 of the launch, and how many of them run whole (the rule of plan_tiled)
static void rag_tiles(const GemmArgs &g, int cus, int64_t *tiles, int64_t *whole)
{
    const int64_t T = ((g.Ra + TILE - 1) / TILE) * ((g.Rb + TILE - 1) / TILE), rem = T % cus;
    *tiles = *whole = T;
    if (g.a_fmt) return;
    if (T < cus) *whole = 0;
    else if (rem != 0 && 2 * rem <= cus && T / cus <= 4) *whole = T - rem;
}

static TileGemm rag_args(const GemmArgs &g)
{
    return TileGemm{g.aq, g.as, g.bq, g.bs, g.C, g.out, g.ld, (int)((g.Ra + TILE - 1) / TILE), (int)((g.Rb + TILE - 1) / TILE)};
}

static hipError_t launch_rag(const GemmArgs &g, int cus, hipStream_t st)
{
    int64_t tiles, whole;
    rag_tiles(g, cus, &tiles, &whole);
    const TileGemm p = rag_args(g);
    const dim3 grid((unsigned)cus);
#define MXFP4_RAG(O, A, F) \
    hipLaunchKernelGGL((gemm_tile_rag_kernel<O, A, F>), grid, dim3(256), 0, st, p, g.Ra, g.Rb, (int)whole)
    if (g.a_fmt) {
        if (!g.out_fp32) MXFP4_RAG(false, false, 1);
        else if (g.accumulate) MXFP4_RAG(true, true, 1);
        else MXFP4_RAG(true, false, 1);
    } else {
        if (!g.out_fp32) MXFP4_RAG(false, false, 0);
        else if (g.accumulate) MXFP4_RAG(true, true, 0);
        else MXFP4_RAG(true, false, 0);
    }
#undef MXFP4_RAG
    return hipGetLastError();
}

// Which kernels a GEMM is cut into (host logic only: no device is touched; cus = compute units of the device).
// Whole 256 x 256 tiles run on the tiled kernel, except where that would leave compute units idle (E2M1 operands):
//   * fewer tiles than compute units: 256 x 128 tiles (twice as many);
//   * a last round of tiles at most half full behind at most four whole rounds: the whole rounds run on 256 x 256
//     tiles and, in the same launch, the tiles of the last round as twice as many 256 x 128 tiles (GEMM_TILED_256_TAIL_128, main_tiles = the tiles of
//     the whole rounds);
//   * a column count in whole 128s but not 256s: 256 x 128 tiles throughout.
// Ragged row or column counts: the 256-aligned interior as above, the right and bottom edge strips (less than one
// tile wide) and everything else as GEMM_ANY (see launch_any).
static void plan_tiled(const GemmArgs &g, int64_t r0, int64_t rows, int64_t cols, int64_t cus, GemmPlan &plan)
{
    auto add = [&](int kind, int64_t main_tiles) {
        plan.part[plan.n++] = GemmPart{kind, r0, rows, 0, cols, main_tiles};
    };
    if (g.a_fmt) return add(GEMM_TILED_256, 0);
    const int64_t T = (rows / TILE) * (cols / TILE);
    if (T < cus) return add(GEMM_TILED_128, 0);
    // (measured: 2 to 5 % on one to three and a half rounds; with more whole rounds in front the second pipeline fill
    // costs as much as the halves save)
    const int64_t rem = T % cus;
    if (rem != 0 && 2 * rem <= cus && T / cus <= 4) return add(GEMM_TILED_256_TAIL_128, T - rem);
    add(GEMM_TILED_256, 0);
}

GemmPlan plan_gemm(const GemmArgs &g, int cus)
{
    GemmPlan plan;
    plan.n = 0;
    if (tile_eligible(g)) {
        plan_tiled(g, 0, g.Ra, g.Rb, cus, plan);
    } else if (tile_eligible(g, TILE / 2)) {
        plan.part[plan.n++] = GemmPart{GEMM_TILED_128, 0, g.Ra, 0, g.Rb, 0};
    } else {
        const int64_t ra = g.Ra / TILE * TILE, rb = g.Rb / TILE * TILE;
        // (the interior starts at offset 0 of every array, so it keeps the alignment of the whole problem; the
        // any-shape kernel asks none of the strips' output pointers)
        if (ra > 0 && rb > 0 && tile_eligible(sub_block(g, 0, ra, 0, rb))) {
            plan_tiled(g, 0, ra, rb, cus, plan);
            if (g.Rb > rb) plan.part[plan.n++] = GemmPart{GEMM_ANY, 0, g.Ra, rb, g.Rb - rb, 0};
            if (g.Ra > ra) plan.part[plan.n++] = GemmPart{GEMM_ANY, ra, g.Ra - ra, 0, rb, 0};
        } else {
            plan.part[plan.n++] = GemmPart{GEMM_ANY, 0, g.Ra, 0, g.Rb, 0};
        }
    }
    return plan;
}

// Estimated microseconds, on the scale of edge_cost (a launch behind another costs 4 us).  A round of 256 x 256 tiles
// takes 1.63 us (MXFP8: 1.9) per stage and 4.5 us, one of 256 x 128 tiles 0.9 us and 3 us.
static double wide_round(const GemmArgs &g) { return (g.a_fmt ? 14.8 : 6.35) * (double)g.C / 1000.0 + 4.5; }
static double narrow_round(const GemmArgs &g) { return 3.5 * (double)g.C / 1000.0 + 3.0; }
static double rounds_of(int64_t tiles, int cus) { return (double)((tiles + cus - 1) / cus); }

static double plan_cost(const GemmArgs &g, const GemmPlan &plan, int cus)
{
    double us = 4.0 * (plan.n - 1);
    for (int i = 0; i < plan.n; ++i) {
        const GemmPart &p = plan.part[i];
        const int64_t tiles = (p.rows / TILE) * (p.cols / TILE);
        if (p.kind == GEMM_TILED_256) us += rounds_of(tiles, cus) * wide_round(g);
        else if (p.kind == GEMM_TILED_128) us += rounds_of((p.rows / TILE) * (p.cols / (TILE / 2)), cus) * narrow_round(g);
        else if (p.kind == GEMM_TILED_256_TAIL_128) us += rounds_of(p.main_tiles, cus) * wide_round(g) + narrow_round(g);
        else us += any_route(sub_block(g, p.r0, p.rows, p.c0, p.cols)).us;
    }
    return us;
}

// The same of moved-back tiles (rows that are not whole cache lines apart: every 128-byte piece is two line requests, of which the narrow
// tile has half as many again per product)
static bool split_lines(const GemmArgs &g) { return (g.a_fmt ? g.C : g.C / 2) % 128 != 0; }
static double rag_wide_round(const GemmArgs &g) { return wide_round(g) * (split_lines(g) ? 1.2 : 1.05); }
static double rag_narrow_round(const GemmArgs &g) { return narrow_round(g) * (split_lines(g) ? 1.3 : 1.05); }

static double rag_cost(const GemmArgs &g, int cus)
{
    if (!rag_eligible(g)) return NO_ROUTE;
    int64_t tiles, whole;
    rag_tiles(g, cus, &tiles, &whole);
    return rounds_of(whole, cus) * rag_wide_round(g) + rounds_of(2 * (tiles - whole), cus) * rag_narrow_round(g) + 1.0;
}

// How two products share a launch of gemm_tile_rag_pair_kernel: tile shapes and split of the chip with the lowest estimate.
struct RagPairChoice {
    int n0, narrow0, narrow1;
    double us;
};
static RagPairChoice choose_rag_pair(const GemmArgs &g0, const GemmArgs &g1, int cus)
{
    RagPairChoice best{0, 0, 0, NO_ROUTE};
    if (cus != NUM_CUS || g0.a_fmt || g1.a_fmt || !g1.out_fp32 || !rag_eligible(g0) || !rag_eligible(g1)) return best;
    if (tile_eligible(g0, TILE / 2) && tile_eligible(g1, TILE / 2)) return best;  // (whole tiles: the launches for these)
    auto tiles = [](const GemmArgs &g) { return ((g.Ra + TILE - 1) / TILE) * ((g.Rb + TILE - 1) / TILE); };
    // Tiles of 1.4 times the outputs' area, narrow outputs for the most part: what is done twice takes what sharing the launch gives.  15 such
    // layers of M x N x K took the same as on gemm_edge_kernel on average (2496 x 8704 x 544 39.5 / 30.2 us, 4032 x 10400 x 544 63 / 58, 8416 x 14080
    // x 288 73 / 86), the others 0.85 times.
    auto area = [&](const GemmArgs &g) { return (double)tiles(g) * TILE * TILE / ((double)g.Ra * (double)g.Rb); };
    if (area(g0) + area(g1) >= 2 * 1.4) return best;
    for (int n0 = 1; n0 < 32; ++n0)
        for (int shapes = 0; shapes < 4; ++shapes) {
            const int narrow0 = shapes & 1, narrow1 = shapes >> 1;
            const double a = rounds_of(tiles(g0) << narrow0, 8 * n0) * (narrow0 ? rag_narrow_round(g0) : rag_wide_round(g0));
            const double b = rounds_of(tiles(g1) << narrow1, 256 - 8 * n0) * (narrow1 ? rag_narrow_round(g1) : rag_wide_round(g1));
            const double us = (a > b ? a : b) + 1.0;
            if (us < best.us) best = RagPairChoice{n0, narrow0, narrow1, us};
        }
    return best;
}

// How a call runs: its plan, or the whole product as one block on the ragged-shape kernel or on the tiled kernel for
// ragged sizes, whichever is estimated to take least.  The plan loses with too few 256 x 128 tiles for the chip (512 x 4096
// x 4096: 14.5 us on 64 tiles, 11.1 us on 128 x 64 ones; in MXFP8, which has no narrow tile, 41.8 and 17.9), where it
// cuts a small product into several launches (300 x 520 x 1024: 15.4 us in three, 4.8 us in one) and where strips beside a
// large interior cost a launch and a poorly filled chip (4010 x 6144 x 4096: 68 us, 60 in one).
// Whole 128s of columns but not 256s: the estimates of 256 x 128 tiles throughout and of 256 x 256 ones moved back lie within
// a few per cent of each other, and decide except for a bf16 output and C < 2048.  Where they prefer the moved-back tiles
// (430 sizes on two cards), these take on average, against the others: bf16 1.04 times as long for C < 2048 (14848 x 3456 x
// 1024 50.8 us, 42.8), 1.01 at 2048, 0.97 beyond; fp32 0.98 at every C.
static GemmRoute choose_route(const GemmArgs &g, const GemmPlan &plan, int cus)
{
    GemmRoute c = any_route(g);
    if (plan.n != 1 || plan.part[0].kind != GEMM_ANY) {
        const double us = plan_cost(g, plan, cus);
        if (us <= c.us || c.kind == ROUTE_ANY_SHAPE) c = GemmRoute{ROUTE_BLOCKS, us};
    }
    const bool narrow = plan.n == 1 && plan.part[0].kind == GEMM_TILED_128 && !g.out_fp32 && g.C < 2048;
    const double rag = narrow ? NO_ROUTE : rag_cost(g, cus);
    if (rag < c.us) c = GemmRoute{ROUTE_RAGGED_TILED, rag};
    return c;
}

GemmRoute route_gemm(const GemmArgs &g, int cus) { return choose_route(g, plan_gemm(g, cus), cus); }

hipError_t launch_gemm(const GemmArgs &g, hipStream_t st)
{
    const int cus = device_cus();
    const GemmPlan plan = plan_gemm(g, cus);
    const GemmRoute route = choose_route(g, plan, cus);
    if (route.kind >= ROUTE_EDGE_64 && route.kind <= ROUTE_EDGE_256)
        return launch_edge(g, nullptr, route.kind - ROUTE_EDGE_64, st);
    if (route.kind == ROUTE_RAGGED_TILED) return launch_rag(g, cus, st);
    for (int i = 0; i < plan.n; ++i) {
        const GemmPart &p = plan.part[i];
        const GemmArgs h = sub_block(g, p.r0, p.rows, p.c0, p.cols);
        hipError_t e;
        if (p.kind == GEMM_ANY)
            e = launch_any(h, st);
        else if (p.kind == GEMM_TILED_128)
            e = launch_tiled_f<0, 2>(h, st);
        else if (p.kind == GEMM_TILED_256_TAIL_128)
            e = launch_tiled_tail(h, p.main_tiles, st);
        else
            e = g.a_fmt ? launch_tiled_f<1, 4>(h, st) : launch_tiled_f<0, 4>(h, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// How gn (narrow tiles first) and gw share a launch of gemm_tile_mix_kernel: the number of rounds of gw that the
// workgroups with a tile of gn add is the one with the lowest estimate.
struct MixChoice {
    int n1, cut;
    double us;
};
static MixChoice choose_mix(const GemmArgs &gn, const GemmArgs &gw, int cus)
{
    MixChoice best{0, 0, NO_ROUTE};
    if (cus != NUM_CUS || gn.a_fmt || gw.a_fmt || !tile_eligible(gn, TILE / 2) || !tile_eligible(gw)) return best;
    const int64_t tn = (gn.Ra / TILE) * (gn.Rb / (TILE / 2)), tw = (gw.Ra / TILE) * (gw.Rb / TILE);
    if (tn > NUM_CUS - 8) return best;
    const int n1 = (int)((tn + 7) / 8), with = 8 * n1, without = NUM_CUS - with;
    for (int extra = 0; extra < 8; ++extra) {
        const int64_t cut = (int64_t)extra * with < tw ? (int64_t)extra * with : tw;
        const double a = narrow_round(gn) + extra * wide_round(gw), b = rounds_of(tw - cut, without) * wide_round(gw);
        const double us = a > b ? a : b;
        if (us < best.us) best = MixChoice{n1, (int)cut, us};
        if (cut == tw) break;
    }
    return best;
}

static hipError_t launch_rag_pair(const GemmArgs &g0, const GemmArgs &g1, int split, hipStream_t st)
{
    const TileGemm p0 = rag_args(g0), p1 = rag_args(g1);
    const int n0 = split & 31, narrow0 = (split >> 5) & 1, narrow1 = (split >> 6) & 1;
#define MXFP4_RAG_PAIR(O0, A1)                                                                                                     \
    hipLaunchKernelGGL((gemm_tile_rag_pair_kernel<O0, A1>), dim3(NUM_CUS), dim3(256), 0, st, p0, g0.Ra, g0.Rb, narrow0, p1, g1.Ra, \
                       g1.Rb, narrow1, n0)
    if (g0.out_fp32) {
        if (g1.accumulate) MXFP4_RAG_PAIR(true, true); else MXFP4_RAG_PAIR(true, false);
    } else {
        if (g1.accumulate) MXFP4_RAG_PAIR(false, true); else MXFP4_RAG_PAIR(false, false);
    }
#undef MXFP4_RAG_PAIR
    return hipGetLastError();
}

static hipError_t launch_mix(const GemmArgs &gn, const GemmArgs &gw, int n1, int cut, hipStream_t st)
{
    const TileGemm pn = tile_args(gn, TILE / 2), pw = tile_args(gw);
#define MXFP4_MIX(ON, AN, OW, AW) \
    hipLaunchKernelGGL((gemm_tile_mix_kernel<ON, AN, OW, AW>), dim3(NUM_CUS), dim3(256), 0, st, pn, pw, n1, cut)
    // (one of the two, problem 0 of the pair, never accumulates)
    if (gn.accumulate) {
        if (gw.out_fp32) MXFP4_MIX(true, true, true, false); else MXFP4_MIX(true, true, false, false);
    } else if (gw.accumulate) {
        if (gn.out_fp32) MXFP4_MIX(true, false, true, true); else MXFP4_MIX(false, false, true, true);
    } else if (gn.out_fp32) {
        if (gw.out_fp32) MXFP4_MIX(true, false, true, false); else MXFP4_MIX(true, false, false, false);
    } else {
        if (gw.out_fp32) MXFP4_MIX(false, false, true, false); else MXFP4_MIX(false, false, false, false);
    }
#undef MXFP4_MIX
    return hipGetLastError();
}

// How two products (g0 without accumulation) that do not depend on each other run: side by side when both fit the tiled
// kernel and together fill the chip; otherwise by estimate.
GemmPairRoute route_gemm_pair(const GemmArgs &g0, const GemmArgs &g1, int cus)
{
    GemmPairRoute r{PAIR_APART, 0, 0, 0};
    // (the split below counts on 8 XCDs of 32 compute units each)
    // Formats: both problems MXFP4 (every combination of output types); or the second, or both, MXFP8 with the
    // output types of a backward pass (bf16 from problem 0, fp32 from problem 1): the stage-wise recipes of Table 1.
    const bool fmt_ok = g0.a_fmt == g0.b_fmt && g1.a_fmt == g1.b_fmt && (g0.a_fmt == 0 || g1.a_fmt == 1) &&
                        (g1.a_fmt == 0 || (!g0.out_fp32 && g1.out_fp32));
    if (!g0.accumulate && fmt_ok && tile_eligible(g0) && tile_eligible(g1) && cus == NUM_CUS) {
        const TileGemm p0 = tile_args(g0), p1 = tile_args(g1);
        const int64_t t0 = (int64_t)p0.tiles_m * p0.tiles_n, t1 = (int64_t)p1.tiles_m * p1.tiles_n;
        // (an E4M3 element costs the matrix unit twice the time of an E2M1 element)
        const double w0 = (double)t0 * (double)g0.C * (g0.a_fmt ? 2.0 : 1.0);
        const double w1 = (double)t1 * (double)g1.C * (g1.a_fmt ? 2.0 : 1.0);
        int n0 = (int)(32.0 * w0 / (w0 + w1) + 0.5);  // workgroups per XCD for g0, in proportion to the work
        n0 = n0 < 1 ? 1 : (n0 > 31 ? 31 : n0);
        // worth it only if both shares have enough tiles to keep their CUs busy
        if (t0 >= (int64_t)n0 * 8 && t1 >= (int64_t)(32 - n0) * 8) {
            r.kind = PAIR_SIDE_BY_SIDE;
            r.n = n0;
            return r;
        }
    }
    // Otherwise by estimate: one after the other, few narrow tiles beside many wide ones, or both on the ragged-shape
    // kernel, the longer contraction first (ragged widths, small layers: a step of 2048 x 3072 x 768 went from 50 to 37 us).
    if (!g0.accumulate && g0.a_fmt == g1.a_fmt && edge_eligible(g0) && edge_eligible(g1)) {
        const EdgeChoice both = choose_edge(g0, &g1);
        const MixChoice mix1 = choose_mix(g1, g0, cus), mix0 = choose_mix(g0, g1, cus);
        const MixChoice mix = mix1.us <= mix0.us ? mix1 : mix0;
        const double apart = route_gemm(g0, cus).us + route_gemm(g1, cus).us + 4.0;
        const RagPairChoice rag = choose_rag_pair(g0, g1, cus);
        // (0.95: of long products the split's estimate is worth less than that, 8672 x 7328 x 10016 took 859 us in one launch, 794 apart; 0.98: of
        // 35 layers nearer to the ragged-shape kernel's estimate 8 were slower, 8448 x 15744 x 320 113 us, 92 on that)
        if (rag.us < 0.95 * apart && rag.us < 0.98 * both.us && rag.us < mix.us)
            r = GemmPairRoute{PAIR_EDGE, 0, EDGE_MOVED_BACK, rag.n0 + 32 * rag.narrow0 + 64 * rag.narrow1};
        else if (mix.us < apart && mix.us < both.us)
            r = GemmPairRoute{PAIR_NARROW_BESIDE_WIDE, mix1.us <= mix0.us ? 1 : 0, mix.n1, mix.cut};
        else if (both.us < apart)
            r = GemmPairRoute{PAIR_EDGE, g1.C > g0.C ? 1 : 0, both.tile, 0};
    }
    return r;
}

hipError_t launch_gemm_pair(const GemmArgs &g0, const GemmArgs &g1, hipStream_t st)
{
    const GemmPairRoute r = route_gemm_pair(g0, g1, device_cus());
    if (r.kind == PAIR_SIDE_BY_SIDE) {
        const TileGemm p0 = tile_args(g0), p1 = tile_args(g1);
        dim3 grid(NUM_CUS);
#define MXFP4_PAIR(O0, O1, A1, F0, F1) \
    hipLaunchKernelGGL((gemm_tile_pair_kernel<O0, O1, A1, F0, F1>), grid, dim3(256), 0, st, p0, p1, r.n)
        if (g1.a_fmt) {
            if (g0.a_fmt) {
                if (g1.accumulate) MXFP4_PAIR(false, true, true, 1, 1); else MXFP4_PAIR(false, true, false, 1, 1);
            } else {
                if (g1.accumulate) MXFP4_PAIR(false, true, true, 0, 1); else MXFP4_PAIR(false, true, false, 0, 1);
            }
        } else if (g0.out_fp32) {
            if (!g1.out_fp32) MXFP4_PAIR(true, false, false, 0, 0);
            else if (g1.accumulate) MXFP4_PAIR(true, true, true, 0, 0);
            else MXFP4_PAIR(true, true, false, 0, 0);
        } else {
            if (!g1.out_fp32) MXFP4_PAIR(false, false, false, 0, 0);
            else if (g1.accumulate) MXFP4_PAIR(false, true, true, 0, 0);
            else MXFP4_PAIR(false, true, false, 0, 0);
        }
#undef MXFP4_PAIR
        return hipGetLastError();
    }
    if (r.kind == PAIR_NARROW_BESIDE_WIDE)
        return r.first ? launch_mix(g1, g0, r.n, r.cut, st) : launch_mix(g0, g1, r.n, r.cut, st);
    if (r.kind == PAIR_EDGE && r.n == EDGE_MOVED_BACK) return launch_rag_pair(g0, g1, r.cut, st);
    if (r.kind == PAIR_EDGE) return r.first ? launch_edge(g1, &g0, r.n, st) : launch_edge(g0, &g1, r.n, st);
    hipError_t e = launch_gemm(g0, st);
    if (e != hipSuccess) return e;
    return launch_gemm(g1, st);
}

}  // namespace mxfp4
