// Host build of the prefill tile arithmetic (csrc/tile_plan.h) for tests/test_tile_plan.py.
#include "tile_plan.h"

extern "C" {

// 0 if the tiles of c tokens are 1 .. kTileM rows each, begin on multiples of 32, follow one
// another from 0 to c, differ by at most one block of 32, and tile_of_row finds each from its
// first and last row; else 1 + the first tile for which that is not so.
int check_rows(int c)
{
    const int m = moe::tiles_of(c), blocks = (c - 1) / 32 + 1;
    int next = 0;
    for (int mt = 0; mt < m; ++mt) {
        const int r0 = moe::tile_row(c, mt), r1 = moe::tile_row(c, mt + 1), h = (r1 - r0 + 31) / 32;
        if (r0 != next || r0 % 32 || r1 <= r0 || r1 - r0 > moe::kTileM || h < blocks / m || h > blocks / m + 1 ||
            moe::tile_of_row(c, r0) != mt || moe::tile_of_row(c, r1 - 1) != mt)
            return 1 + mt;
        next = r1;
    }
    return next == c ? 0 : 1 + m;
}

void plan(int U, int nsteps, int slots, int planes, int maxparts, int pairs, int xcd, int *out)
{
    const int r = moe::tile_plan(U, slots, xcd, 1).units % slots;
    int key = moe::split_key(r, nsteps, slots, planes, maxparts, pairs, 1);
    for (int s = 2; s <= moe::kMaxSplit; ++s) {
        const int k = moe::split_key(r, nsteps, slots, planes, maxparts, pairs, s);
        if (k < key) key = k;
    }
    const moe::TilePlan p = moe::tile_plan(U, slots, xcd, key % moe::kMaxSplit + 1);
    out[0] = p.u0;
    out[1] = p.units;
    out[2] = p.full;
    out[3] = p.s;
}

int planes_of(int T) { return moe::max_planes(T); }

size_t offset_of(int row, int K, int at) { return moe::operand_offset(row, K, at); }

int xcd_of(int U, int u) { return moe::xcd_of_tile(U, u); }

}  // extern "C"
