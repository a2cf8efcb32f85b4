// Device code shared by the quantiser kernels (MXFP4 in quantize.hip, MXFP8 in quantize_fp8.hip): the counter
// hash, one block's rotation and maximum in registers, bf16 widening, and the column-wise workgroup tile.
// Everything sits in an unnamed namespace: each translation unit gets its own copy.
#pragma once
#include "mxfp4_internal.h"

namespace mxfp4 {
namespace {

constexpr int HAD_NONE = 0, HAD_DET = 1, HAD_RANDSIGN = 2, HAD_DET16 = 3, HAD_RANDSIGN16 = 4;
constexpr int RND_RNE = 0, RND_SR = 1;

// ---- counter hash: stateless 32-bit mixer applied to (seed, index) -----------------
struct RngKey {
    uint32_t seed_lo_mul;  // low seed word times the odd constant
    uint32_t seed_hi_mix;  // mixed high seed word
};

__host__ __device__ __forceinline__ uint32_t mix32(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x9E3779B9u;
    x ^= x >> 15;
    x *= 0xBB67AE85u;
    x ^= x >> 16;
    return x;
}

__host__ __device__ __forceinline__ uint32_t rand32(RngKey k, uint64_t idx)
{
    return mix32(mix32((uint32_t)idx + k.seed_lo_mul) ^ (uint32_t)(idx >> 32) ^ k.seed_hi_mix);
}

// The same for element i (0..31) of a block, but for the last step (x ^= x >> 16): low = low index word of its first element plus
// seed_lo_mul, mixed_high = h ^ h >> 16 with h = high index word ^ seed_hi_mix.  (Two such steps with an xor between them undo each other:
// what ends the first mix32 and what begins the second become one xor.)
__device__ __forceinline__ uint32_t rand32_in_block(uint32_t low, uint32_t mixed_high, int i)
{
    uint32_t x = low + (uint32_t)i;
    x ^= x >> 16;
    x *= 0x9E3779B9u;
    x ^= x >> 15;
    x *= 0xBB67AE85u;
    x ^= mixed_high;
    x *= 0x9E3779B9u;
    x ^= x >> 15;
    return x * 0xBB67AE85u;
}

RngKey make_key(uint64_t seed)
{
    RngKey k;
    k.seed_lo_mul = (uint32_t)seed * 0x9E3779B9u;
    k.seed_hi_mix = mix32((uint32_t)(seed >> 32) ^ 0x6A09E667u);
    return k;
}

// the +-1 diagonal of the random-sign rotation: a function of the base seed alone
uint32_t sign_mask_of(uint64_t seed) { return rand32(make_key(seed & SEED_BASE_MASK), 0xFFFFFFFFFFFFFFFFull); }

// ---- one block in registers ---------------------------------------------------------
template <int N>
__device__ __forceinline__ void butterflies(float (&v)[32])
{
#pragma unroll
    for (int h = 1; h < N; h <<= 1) {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            if ((i & h) == 0) {
                float a = v[i], b = v[i + h];
                v[i] = a + b;
                v[i + h] = a - b;
            }
        }
    }
}

// Stochastic rounding of v to an E2M1 code under the scale 2^(sb - 127), in the top four bits of the result (sign in bit 31).  With
// a = min(|v| / scale, 6) between two neighbours of the grid and f its distance from the lower one in grid steps, the magnitude goes up
// iff u < f, u = (2 R + 1) 2^-24, R = r >> 9.  As integers: let y be the code of the lower neighbour times 2^28 plus f 2^28, rounded up.
// 16 (2 R + 1) < f 2^28 holds iff y's fraction is at least 32 R + 17, i.e. iff adding 2^28 - 32 R - 17 carries into the code.  Below 2 the
// grid is uniform and y is a 2^29; from 1 upwards y is a's bit pattern shifted (a grid step is half an octave), which is the smaller
// of the two from 2 on.  (|v| / scale is below 8, so a 2^29 fits 32 bits without the clamp.)
// The kernels that round stochastically are bound by their vector instructions: 23 per element and block (29 with loads, stores and addresses); 30
// with a comparison to select y, sign and code packed apart and the whole hash, 42 with the rounding decided in floating point.  With four waves per
// SIMD an xor, a sum or a shift takes 2.4 clocks of it, the others here (products of 32 bits as much as a fused shift or a conversion) 4.2: 23 are
// 38 us of 16384 x 4096, 29 are 46.  That tensor, us, with 42, 30 and 23: row-wise 69, 61, 53, column-wise 76, 61, 57, both 149, 119, 104 (29, 39 and
// 53 rounding to nearest).
// hash: the counter hash before its last step, r = hash ^ hash >> 16
__device__ __forceinline__ uint32_t sr_code(float v, int to_2_29, uint32_t hash)
{
    const float a = __builtin_fabsf(__builtin_ldexpf(v, to_2_29));
    const uint32_t low = (uint32_t)__builtin_ceilf(a);
    const float clamped = __builtin_amdgcn_fmed3f(a, 0x1p29f, 0x1.8p31f);
    const uint32_t high = (__float_as_uint(clamped) << 6) + 0xA0000000u;  // 2^29 -> 2 << 28, ... 6 2^29 -> 7 << 28
    const uint32_t y = (low < high ? low : high) + ((~(hash >> 4 ^ hash >> 20) & 0x0FFFFFE0u) | 15u);
    return __float_as_uint(__builtin_copysignf(__uint_as_float(y), v));
}

// Optional sign flips and rotation of one block, in place (App. A.2).
template <int HAD>
__device__ __forceinline__ void rotate_block(float (&v)[32], uint32_t sign_mask)
{
    if (HAD == HAD_RANDSIGN || HAD == HAD_RANDSIGN16) {  // the block's 32-entry diagonal, whatever the rotation size
#pragma unroll
        for (int i = 0; i < 32; ++i)
            v[i] = __uint_as_float(__float_as_uint(v[i]) ^ (((sign_mask >> i) & 1u) << 31));
    }
    if (HAD == HAD_DET || HAD == HAD_RANDSIGN) {
        butterflies<32>(v);
        const float c = __uint_as_float(0x3E3504F3u);  // 2^-2.5 rounded to fp32
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = v[i] * c;
    } else if (HAD == HAD_DET16 || HAD == HAD_RANDSIGN16) {
        butterflies<16>(v);
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = v[i] * 0.25f;
    }
}

// Bit pattern of the block's largest magnitude.  V_MAXIMUM3_F32 (two new values per instruction, |.| as source
// modifiers) returns NaN if any input is NaN, so a NaN or an infinity anywhere in the block shows as an exponent
// field of 255, as in a comparison of the bit patterns.
__device__ __forceinline__ uint32_t amax_bits(const float (&v)[32])
{
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 32; i += 2)
        m = __builtin_elementwise_maximum(
            __builtin_elementwise_maximum(__builtin_fabsf(v[i]), __builtin_fabsf(v[i + 1])), m);
    return __float_as_uint(m) & 0x7FFFFFFFu;
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// 32 contiguous bf16 (four 16-byte words) widened to fp32
__device__ __forceinline__ void widen(const uint4 (&raw)[4], float (&v)[32])
{
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[8 * j + 0] = bf16_lo(raw[j].x);
        v[8 * j + 1] = bf16_hi(raw[j].x);
        v[8 * j + 2] = bf16_lo(raw[j].y);
        v[8 * j + 3] = bf16_hi(raw[j].y);
        v[8 * j + 4] = bf16_lo(raw[j].z);
        v[8 * j + 5] = bf16_hi(raw[j].z);
        v[8 * j + 6] = bf16_lo(raw[j].w);
        v[8 * j + 7] = bf16_hi(raw[j].w);
    }
}

// FP4 codes of one rotated block under the scale that follows from the shared maximum `amax` (bit
// pattern): eq. (1) with the OCP scale rule.  idx0: linear index of element 0 in the quantised output
// (stochastic rounding counter).
template <int RND>
__device__ __forceinline__ void encode_scaled(const float (&v)[32], uint32_t amax, RngKey key, uint64_t idx0,
                                              uint4 &codes, uint32_t &scale_byte)
{
    uint32_t eb = amax >> 23;
    bool bad = (eb == 255u);
    uint32_t sb = eb > 2u ? eb - 2u : 0u;  // eb <= 254 here, so sb <= 252
    scale_byte = bad ? 0xFFu : sb;

    uint32_t w[4];
    if (RND == RND_RNE) {
        // The converter divides by 2^(exponent field of `scale` - 127), rounds to nearest
        // even on the E2M1 grid and saturates at 6; it writes one byte (two codes) per issue.
        float scale = __uint_as_float(sb << 23);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t r = 0;
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * j + 0], v[8 * j + 1], scale, 0);
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * j + 2], v[8 * j + 3], scale, 1);
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * j + 4], v[8 * j + 5], scale, 2);
            r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * j + 6], v[8 * j + 7], scale, 3);
            w[j] = r;
        }
    } else {
        const int to_2_29 = 29 + 127 - (int)sb;
        // (a block starts at a multiple of 32: its elements share the index's high word)
        const uint32_t low = (uint32_t)idx0 + key.seed_lo_mul, high = (uint32_t)(idx0 >> 32) ^ key.seed_hi_mix;
        const uint32_t mixed = high ^ high >> 16;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t r = 0;
#pragma unroll
            for (int e = 7; e >= 0; --e)
                r = __builtin_amdgcn_alignbit(r, sr_code(v[8 * j + e], to_2_29, rand32_in_block(low, mixed, 8 * j + e)), 28);
            w[j] = r;
        }
    }
    codes = bad ? make_uint4(0, 0, 0, 0) : make_uint4(w[0], w[1], w[2], w[3]);
}

// Code store.  streaming: for tensors larger than the 256 MB last-level cache the output cannot stay cached
// for the GEMM anyway, and marking the stores non-temporal is worth 3-8 % there (measured); smaller tensors
// keep ordinary stores so that the GEMM finds its operands in cache.
__device__ __forceinline__ void store_codes(uint4 *p, uint4 v, int streaming)
{
    if (streaming) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store((u32x4){v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(p));
    } else {
        *p = v;
    }
}

// ---- column-wise workgroup tile: a row block of 32 per wave x 128 columns (2 per lane) ----
constexpr int CT_COLS = 128;
constexpr int RAW_PITCH = 272;  // bytes per parked row: 256 + 16, so that the 16-byte reads below (16 lanes =
                                // 4 rows x 4 blocks per issue) and the dword writes touch every bank once

// Orders the LDS accesses of one wave (which the hardware performs in program order) for the compiler too.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace
}  // namespace mxfp4
