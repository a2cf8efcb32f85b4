// Which products on the ragged-shape kernel's 64 x 64 and 128 x 64 tiles run as the kernels for few outputs (32 x 32 tiles) and for short rows
// (plain arithmetic, free of HIP types).
#pragma once
#include <stdint.h>

namespace mxfp4 {

struct EdgeProduct {
    int64_t Ra, Rb;
    int64_t row_bytes;  // of codes
    int64_t pitch;      // bytes from one row of the output to the next
    bool e4m3, fp32, accumulate;
};

constexpr int64_t edge_stages(const EdgeProduct &p) { return (p.row_bytes + 127) / 128; }
constexpr int64_t edge_tiles(const EdgeProduct &p, int tm, int tn) { return (p.Ra + tm - 1) / tm * ((p.Rb + tn - 1) / tn); }

// Whether 32 x 32 tiles, `tiles` of them in the launch, are the faster ones for a product.  Time on them over time on 64 x 64 ones:
//   * whole stages (rows of whole 128 bytes): up to 256 tiles MXFP4 0.9 at one stage, 0.83 at 3, 0.73 at 6 (MXFP8 0.95, 0.85, 0.78), up to 512
//     tiles 0.97, 0.95, 0.86 from two stages on (0.98, 0.98, 0.9), 1.02 to 1.05 at one;
//   * a ragged last stage, whose scale bytes are moved before anything is multiplied, costs them 0.3 us: up to 256 tiles 1.03 to 1.08 at one stage,
//     0.97 to 1.0 at two, 0.9 at four (MXFP8 1.08 to 1.14, 1.02 to 1.06, 0.95; 0.97 to 1.0 at three), up to 512 tiles 1.0 at four, 0.93 at
//     five (MXFP8 1.03 at six, 1.0 at eight).
// More than 512 tiles, over two workgroups per compute unit: 0.9 to 1.7.
constexpr bool small_gains(const EdgeProduct &p, int64_t tiles)
{
    if (tiles > 512) return false;
    const int64_t stages = edge_stages(p);
    if (p.row_bytes % 128 == 0) return tiles <= 256 || stages >= 2;
    return tiles <= 256 ? stages >= (p.e4m3 ? 3 : 2) : stages >= (p.e4m3 ? 8 : 5);
}
// Of the products (or pairs) on 64 x 64 tiles, those on 32 x 32 ones: the number of these, else 0.
constexpr int small_tiles(const EdgeProduct &p0, const EdgeProduct *p1)
{
    const int64_t tiles = edge_tiles(p0, 32, 32) + (p1 ? edge_tiles(*p1, 32, 32) : 0);
    return small_gains(p0, tiles) && (!p1 || small_gains(*p1, tiles)) ? (int)tiles : 0;
}

// Whether 128 x 64 tiles run as gemm_short_kernel: at most two stages, and output rows that are not whole cache lines apart, or more
// than 4096 tiles.  Such rows it stores in longer pieces: 2048 x 3000 x 288 bf16 10.2 us on 128 x 256 tiles, 7.5 on this, added to in
// fp32 16.5, 11.4; 512 x 10000 x 512 9.1, 7.1.  Where each row starts a line the other kernels' stores are as good, and few tiles are
// done sooner there: 2048 x 4096 x 512 8.2, 9.6 (1024 tiles), 4096 x 4096 x 512
// 14.1, 14.9 (2048 tiles), 512 x 7040 x 512 fp32 6.6, 8.0; many overlap here: 8192 x 8192 x 512 fp32 69.9, 62.6, 12526 x 9728 x 256 80, 55.
// An fp32 product alone stays on the other kernels' tiles, too,
//   * with two stages and 769 to 1024 tiles, of which 768 run at once (the last round nearly empty costs more than its rows gain): 608 x 10368 x 512
//     10.2 us, on this 11.6, MXFP8 1152 x 5960 x 192 10.7, 11.7; rows in no whole 16 bytes only if it is added to (1280 x 5764 x 480 1.1
//     times as long);
//   * added to with at most 512 tiles, which the others hold at once: 1920 x 1360 x 64 6.9, 8.0, 5369 x 656 x 32 7.3, 8.4, 1280 x 2536 x 480 1.07
//     times as long.
constexpr bool runs_short(const EdgeProduct &p0, const EdgeProduct *p1)
{
    auto fits = [](const EdgeProduct &p) { return edge_stages(p) <= 2 && (p.pitch % 128 != 0 || edge_tiles(p, 128, 64) > 4096); };
    if (!fits(p0) || (p1 && !fits(*p1))) return false;
    if (p1 || !p0.fp32) return true;
    const int64_t tiles = edge_tiles(p0, 128, 64);
    if (edge_stages(p0) == 2 && tiles > 768 && tiles <= 1024 && (p0.accumulate || p0.pitch % 16 == 0)) return false;
    return !p0.accumulate || tiles > 512;
}

}  // namespace mxfp4
