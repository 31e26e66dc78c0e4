// Which tile of C and which K slice a workgroup takes.  Plain C++17 whose functions are constexpr, so that the kernels, the host code
// that launches them and a test built with the host compiler run the same text.
#pragma once

#include <stdint.h>

namespace peak {

// Division by a number that the host knows: 2^32 over it, rounded down (2^32 - 1 for 1); the quotient it gives is one short at most.
struct Divisor {
    uint32_t d, r;
};
static constexpr Divisor divisor(int d) { return Divisor{(uint32_t)d, d == 1 ? 0xFFFFFFFFu : (uint32_t)(((uint64_t)1 << 32) / (uint64_t)d)}; }

// (By the host's reciprocals: a workgroup works out its tile before it can ask for anything.  The compiler's four divisions, and one
// in 64 bits for a K rotation that most launches do not have, took 0.1 to 0.3 us of each launch: fp32 256^3 NN 4.68 us and 4.37,
// 512^3 5.91 and 5.57, 300^3 TT 5.01 and 4.55; bf16 512x4096x1024 NT 7.68 and 7.55, 100x4096x4096 11.10 and 10.97, 2048x2048x512 8.47 and 8.33.)
static constexpr int quotient(uint32_t n, const Divisor &by)
{
    const uint32_t q = (uint32_t)((uint64_t)n * by.r >> 32);
    return (int)(n - q * by.d >= by.d ? q + 1 : q);
}

// Tile order (the paper's Block-Swizzle, made XCD-aware): consecutive workgroup
// ids go round-robin to the 8 XCDs, each with its own L2.  Give every XCD a
// contiguous run of the band-ordered tile list, so the tiles an XCD works on at
// one time share A row panels and B column panels in that L2.  A plan that splits
// K orders (slice, tile) as one list: with few tiles an XCD then holds one stretch
// of K of many tiles, where dealing out each slice by itself gave it the same few
// tiles in every slice and nothing that two of them share (bf16 1768x160x7784 TN
// in 6 slices 22.6 -> 16.3 us, f16 640x448x16512 NN in 12 30.5 -> 23.1, 1280x1144x18248
// NN in 5 77.9 -> 67.2; 51 split plans 7 % with warm operands, 5 % from HBM).
static constexpr int order_of_block(int t, int total)
{
    const int xcd = t & 7, idx = t >> 3;
    const int base = total >> 3, rem = total & 7;
    return xcd * base + (xcd < rem ? xcd : rem) + idx;
}

// The tiles of C in bands of group_m tile rows (the last band may have fewer), down a band's rows first.  Args has tiles_m, tiles_n,
// group_m and the divisors by_tiles (tiles_m * tiles_n), by_band (tiles of a band), by_group and by_last (rows of a band and of the last one).
template <class Args>
static constexpr void set_tile_order(Args &a, int tiles_m, int tiles_n, int group_m)
{
    a.tiles_m = tiles_m; a.tiles_n = tiles_n;
    a.group_m = group_m;
    a.by_tiles = divisor(tiles_m * tiles_n);
    a.by_band = divisor(group_m * tiles_n);
    a.by_group = divisor(group_m);
    a.by_last = divisor(tiles_m % group_m ? tiles_m % group_m : group_m);
}
template <class Args>
static constexpr void tile_in_order(const Args &p, int L, int &tm, int &tn)
{
    const int g = quotient((uint32_t)L, p.by_band);
    const int first = g * p.group_m, left = p.tiles_m - first;
    const bool last = left < p.group_m;
    const int gsz = last ? left : p.group_m, w = L - g * (int)p.by_band.d;
    tn = last ? quotient((uint32_t)w, p.by_last) : quotient((uint32_t)w, p.by_group);
    tm = first + w - tn * gsz;
}

}  // namespace peak
