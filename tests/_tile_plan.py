"""The plan of the prefill GEMMs for a routing, as csrc/tile_plan.h and the workspace layout of
csrc/prefill.hip make it (test_tile_plan.py compares this copy with the header), so that a
test can assert which branches its shape reaches."""
XCDS, TILE_M, MAX_SPLIT, MIN_STEPS, SPLIT_STEPS = 8, 256, 16, 4, 4


def max_planes(T):
    return 8 if T < 128 else 4


def split(r, nsteps, slots, planes, maxparts, pairs):
    best, parts = nsteps, 1
    for s in range(2, MAX_SPLIT + 1):
        fits = s <= 4 or r * s <= slots if s <= planes else r * s <= maxparts
        if r == 0 or s * MIN_STEPS > nsteps or not fits:
            continue
        reads = (s - 4) * (1 + pairs // 64) if 4 < s <= planes else 0
        cost = -(-r * s // slots) * (-(-nsteps // s) + SPLIT_STEPS) + reads
        if cost < best:
            best, parts = cost, s
    return parts


def plan(U, nsteps, slots, planes, maxparts, pairs):
    """(first tile, tiles, whole tiles, K parts of the others) of each XCD."""
    out = []
    for x in range(XCDS):
        u0 = U * x // XCDS
        units = U * (x + 1) // XCDS - u0
        s = split(units % slots, nsteps, slots, planes, maxparts, pairs)
        out.append((u0, units, units - units % slots if s > 1 else units, s))
    return out


def prefill_plans(d, f, n, k, T, counts, cus=256):
    """Plans of gate/up and down for `counts` tokens per expert and the recommended workspace."""
    tiles = sum(-(-c // TILE_M) for c in counts)
    planes, slots = max_planes(T), cus // XCDS
    extra = 48 << 20 if T * k >= 64 * n else 0
    part = XCDS * min(T, TILE_M) * 256 * 4
    gu = 0 if T < 16 else min(64, (min(planes, 4) * T * k * d * 4 + extra) // part)
    dn = min(64, extra // part)
    return (plan(tiles * (f // 128), d // 64, slots, 1, gu, T * k),
            plan(tiles * -(-d // 256), f // 64, slots, planes, dn, T * k))
