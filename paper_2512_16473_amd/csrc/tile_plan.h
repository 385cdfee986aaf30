// Work decomposition of a grouped GEMM of prefill, planned on the device from the routing
// (host and device functions: the arithmetic is checked on the CPU).
//
// Expert e's c tokens are cut into m = ceil(c / kTileM) tiles, equal to within a block of
// 32 rows. A GEMM's output tiles, in (expert, N tile, M tile) order with the M tile
// fastest, are dealt out to the XCDs in eight contiguous runs of equal length, so that the
// tiles that share an expert's token rows (and, side by side, a weight tile) run on one
// XCD's L2, whatever the number of experts. On an XCD the work groups (one per CU,
// `slots` of them) take its tiles in rounds; the r tiles of a last, partial round are
// split over K into s parts each, whose fp32 sums a later kernel adds in order. The sums of
// up to `planes` parts of a down tile go to as many planes of the output; otherwise each part
// has a buffer of its own.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace moe {

constexpr int kXcds = 8;
constexpr int kTileM = 256;       // tokens per tile, at most
constexpr int kMaxSplit = 16;     // K parts per split tile
constexpr int kMinPartSteps = 4;  // K steps per part, at least
constexpr int kSplitSteps = 4;    // what a part costs besides its K steps, in K steps

struct TilePlan {
    int u0, units;   // first tile of the XCD's run, its length
    int full;        // tiles done whole; the other units - full are split over K
    int s;           // K parts of a split tile
};

__host__ __device__ inline int tiles_of(int c) { return (c + kTileM - 1) / kTileM; }

// First row of tile mt of an expert with c tokens (mt == tiles_of(c): c). Its ceil(c / 32)
// blocks of 32 rows are spread evenly, so that few padding rows are multiplied: the first
// blocks % tiles tiles hold one block more than the others. (No product of blocks and tiles,
// which passes 32 bits from 5.9 million tokens on.)
__host__ __device__ inline int tile_row(int c, int mt)
{
    const uint32_t blocks = (uint32_t)(c + 31) >> 5, m = tiles_of(c);
    if (m <= 1) return mt ? c : 0;
    const uint32_t q = blocks / m, more = blocks - q * m, t = mt;
    const int row = (int)(t * q + (t < more ? t : more)) * 32;
    return row < c ? row : c;
}
// the tile that holds row r
__host__ __device__ inline int tile_of_row(int c, int r)
{
    const uint32_t blocks = (uint32_t)(c + 31) >> 5, m = tiles_of(c);
    if (m <= 1) return 0;
    const uint32_t q = blocks / m, more = blocks - q * m;
    const uint32_t b = (uint32_t)r >> 5, tall = more * (q + 1);   // blocks of the taller tiles
    const bool in = b < tall;
    return (int)((in ? 0 : more) + (in ? b : b - tall) / (in ? q + 1 : q));
}

// What s parts (1 .. kMaxSplit) of each of r split tiles of nsteps K steps cost, and s: the plan
// takes the s whose key is least. A split costs about as much as a few K steps (prologue,
// fp32 sums), and every plane beyond four one that the combine reads in turn (100 tokens on 8
// experts of d = 1152, f = 2048: 42.6 us with four parts, 43.6 with eight); the parts have to
// fit the planes or the part buffers. More than four planes are for work groups that would
// idle, so the parts are one round (4 tokens on 32 experts top-6 of d = 1152, f = 7680: 172 us
// with two parts, 177 with five in two rounds).
__host__ __device__ inline int split_key(int r, int nsteps, int slots, int planes, int maxparts, int pairs, int s)
{
    constexpr int kNever = 0x7ffffff;
    int cost = nsteps;
    if (s > 1) {
        const int reads = s > 4 && s <= planes ? (s - 4) * (1 + pairs / 64) : 0;
        cost = (r * s + slots - 1) / slots * ((nsteps + s - 1) / s + kSplitSteps) + reads;
        const bool fits = s <= planes ? s <= 4 || r * s <= slots : r * s <= maxparts;
        if (r == 0 || s * kMinPartSteps > nsteps || !fits) cost = kNever;
    }
    return (cost < kNever ? cost : kNever) * kMaxSplit + (s - 1);
}

// XCD xcd's run of U tiles, with the tiles of a last, partial round in s parts.
__host__ __device__ inline TilePlan tile_plan(int U, int slots, int xcd, int s)
{
    TilePlan p;
    p.u0 = (int)((int64_t)U * xcd / kXcds);
    p.units = (int)((int64_t)U * (xcd + 1) / kXcds) - p.u0;
    p.full = s > 1 ? p.units - p.units % slots : p.units;
    p.s = s;
    return p;
}

// Planes of the down output, at most, for T tokens. Short prompts have few down tiles and few
// part buffers or none, so that the planes limit the work groups that read W2: with four, one
// token on f = 14336, d = 384 ran on 8 of them and took 57.9 us, with eight 43.5 (12 groups of
// 128-row tiles: 52.8); 63 tokens on 8 experts of f = 14336, d = 256 82.9 -> 70.0. From 128
// tokens on there are the tiles or the part buffers.
__host__ __device__ inline int max_planes(int T) { return T < 128 ? 8 : 4; }

// The XCD whose run holds tile u of U.
__host__ __device__ inline int xcd_of_tile(int U, int u)
{
    return (int)(((int64_t)kXcds * u + kXcds - 1) / U);
}

// Byte offset of byte `at` of operand row `row` of K bf16 values. (64 bits: the 256 rows of a
// down tile span 4 GiB from K = 8.4 million on.)
__host__ __device__ inline size_t operand_offset(int row, int K, int at)
{
    return (size_t)row * (size_t)K * 2 + (size_t)at;
}

}  // namespace moe
