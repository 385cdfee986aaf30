// Prefill MoE layer: T tokens through one layer with every expert resident.
//
// Steps (each a kernel on one stream):
//   1. router for all T tokens (the batched router kernel);
//   2. grouping: a stable counting sort of the T*k (token, rank) pairs by expert, giving
//      per-expert offsets, the tokens in expert order, each pair's place, and the tile
//      plans of the two GEMMs;
//   3. hidden states rounded to bf16 for the matrix cores (other blocks of the grouping
//      launch: it does not depend on the routing);
//   4. grouped GEMM gate/up: for each expert e, H_e = SiLU(X_e W1_e^T) * (X_e W3_e^T),
//      bf16 MFMA (v_mfma_f32_16x16x32_bf16) with fp32 accumulation, H_e stored bf16; the
//      tiles of a last, partial round of work groups are split over K, and
//   4b. a small kernel adds their parts and applies SiLU * up;
//   5. grouped GEMM down: Y_e = H_e W2_e^T in fp32, the last round split likewise;
//   6. combine: OUT[t] = sum_r w[t][r] * Y[pair(t, r)], in a fixed order, adding the parts
//      of split tiles as it reads them.
//
// Up to a few hundred tokens per expert the GEMMs are bound by reading the expert weights
// from HBM; beyond, by the matrix cores.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "moe_internal.h"
#include "tile_plan.h"

namespace moe {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kGemmThreads = 512;
constexpr int kBK = 64;              // K per stage
constexpr int kTileN = 256;          // weight rows per tile
constexpr int kGuCols = kTileN / 2;  // gate/up: H columns per tile
constexpr int kLdsBytes = 163840;    // all of a CU's LDS
constexpr int kMaxParts = 64;        // part buffers per XCD
constexpr int kStagger = 2;          // K steps between the starts of neighbouring N tiles

__device__ __forceinline__ uint16_t f2bf(float f)
{
    // round to nearest even (inputs are finite)
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// SiLU(g) * u rounded to bf16, within 2.5 fp32 ulps before that rounding. (The hardware's exp2
// of a scaled g and its reciprocal take 2530 instead of 2576 us for 4096 Mixtral-shaped tokens
// and 814 instead of 829 us for 1333 fine-grained ones, but are up to 5e-6 relative off as -g
// grows and flush a sigmoid below 2^-126 to zero.)
__device__ __forceinline__ uint16_t swiglu_bf(float g, float u)
{
    return f2bf(g / (1.0f + expf(-g)) * u);
}

// y = bf16(x) over n8 groups of 8 values; `first`, `stride`: this thread's first group
// and the step between its groups.
__device__ __forceinline__ void cast_bf16(const float *x, uint16_t *y, int64_t n8, int64_t first, int64_t stride)
{
    for (int64_t i = first; i < n8; i += stride) {
        const float4 a = reinterpret_cast<const float4 *>(x)[2 * i];
        const float4 b = reinterpret_cast<const float4 *>(x)[2 * i + 1];
        uint4 o;
        o.x = f2bf(a.x) | ((uint32_t)f2bf(a.y) << 16);
        o.y = f2bf(a.z) | ((uint32_t)f2bf(a.w) << 16);
        o.z = f2bf(b.x) | ((uint32_t)f2bf(b.y) << 16);
        o.w = f2bf(b.z) | ((uint32_t)f2bf(b.w) << 16);
        reinterpret_cast<uint4 *>(y)[i] = o;
    }
}

// Orders the wave's LDS accesses before and after it (the barrier alone orders no memory for
// the compiler; the hardware runs a wave's LDS accesses in order, so this is no instruction).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Block 0: the grouping below. Blocks 1 ..: the hidden states rounded to bf16 for the
// matrix cores (independent of the routing, so the two share one launch).
// Stable counting sort of the pairs p = t*k + r by expert idx[p] (one block): off[e] ..
// off[e+1] is expert e's range, tok the token of each place, pos[p] the place of pair p.
// Each wave owns a run of consecutive pairs: it counts them per expert, the counts are
// scanned over experts and waves, and the wave walks its run again, 64 pairs at a time; a
// pair's place among its expert's in the 64 is the number of lower lanes with the same
// expert, found with one ballot per bit of the id. No barrier inside either walk. (Counting
// earlier pairs in LDS, 1024 pairs per barrier, the launch took 86 us for 10664 pairs and
// 70 us for 8192; now 20 and 19 us, the cast included.)
constexpr int kGroupThreads = 1024;
constexpr int kGroupWaves = kGroupThreads / 64;
struct GroupArgs {
    const int32_t *idx;              // [npairs]
    int npairs, n, k;
    int32_t *off, *toff, *tok, *pos;
    TilePlan *plan;                  // [2][8]: gate/up, down
    int ntiles[2], nsteps[2], maxparts[2], slots, planes;
    const float *x;
    uint16_t *xb;
    int64_t n8;
};
__global__ __launch_bounds__(kGroupThreads) void k_group(GroupArgs g)
{
    if (blockIdx.x > 0) {
        cast_bf16(g.x, g.xb, g.n8, (int64_t)(blockIdx.x - 1) * kGroupThreads + threadIdx.x,
                  (int64_t)(gridDim.x - 1) * kGroupThreads);
        return;
    }
    __shared__ int32_t next[kGroupWaves][MOE_MAX_EXPERTS];   // counts, then the next free place
    __shared__ int2 wsum[MOE_MAX_EXPERTS / 64];              // pairs and tiles of 64 experts
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    for (int i = t; i < kGroupWaves * MOE_MAX_EXPERTS; i += kGroupThreads) next[0][i] = 0;
    __syncthreads();
    const int per = ((g.npairs + kGroupThreads - 1) / kGroupThreads) * 64;   // pairs per wave
    const int p0 = wv * per, p1 = min(p0 + per, g.npairs);
    for (int p = p0 + lane; p < p1; p += 64) atomicAdd(&next[wv][g.idx[p]], 1);
    __syncthreads();
    // scan: thread e < 256 holds expert e (whole waves 0-3)
    int c = 0, pairs = 0, tiles = 0;
    if (t < MOE_MAX_EXPERTS) {
#pragma unroll
        for (int w = 0; w < kGroupWaves; ++w) {   // counts -> exclusive sums over the waves
            const int v = next[w][t];
            next[w][t] = c;
            c += v;
        }
        pairs = c;
        tiles = tiles_of(c);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {        // inclusive sums over the wave's experts
            const int a = __shfl_up(pairs, o, 64), b = __shfl_up(tiles, o, 64);
            if (lane >= o) {
                pairs += a;
                tiles += b;
            }
        }
        if (lane == 63) wsum[wv] = make_int2(pairs, tiles);
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < MOE_MAX_EXPERTS / 64; ++w) total += wsum[w].y;
    if (t < MOE_MAX_EXPERTS) {
        for (int w = 0; w < wv; ++w) {
            pairs += wsum[w].x;
            tiles += wsum[w].y;
        }
        const int first = pairs - c;              // expert t's first place
#pragma unroll
        for (int w = 0; w < kGroupWaves; ++w) next[w][t] += first;
        if (t < g.n) {
            g.off[t] = first;
            g.toff[t] = tiles - tiles_of(c);
            if (t == g.n - 1) {
                g.off[g.n] = pairs;
                g.toff[g.n] = tiles;
            }
        }
    }
    // The plans, by the next four waves: 16 lanes weigh the splits of one (with a thread going
    // through the splits of a plan the launch took 4.7 us for a token of d = 1408, f = 5632, now 3.2).
    static_assert(kMaxSplit == 16 && 2 * kXcds * kMaxSplit == MOE_MAX_EXPERTS, "four waves of 16 lanes a plan");
    if (t >= MOE_MAX_EXPERTS && t < 2 * MOE_MAX_EXPERTS) {
        const int j = (t - MOE_MAX_EXPERTS) / kMaxSplit, q = j / kXcds, xcd = j % kXcds;
        const int U = total * g.ntiles[q], r = tile_plan(U, g.slots, xcd, 1).units % g.slots;
        int key = split_key(r, g.nsteps[q], g.slots, q ? g.planes : 1, g.maxparts[q], g.npairs, t % kMaxSplit + 1);
#pragma unroll
        for (int o = 1; o < kMaxSplit; o <<= 1) key = min(key, __shfl_xor(key, o, 64));
        if (t % kMaxSplit == 0) g.plan[j] = tile_plan(U, g.slots, xcd, key % kMaxSplit + 1);
    }
    __syncthreads();
    int e = p0 + lane < p1 ? g.idx[p0 + lane] : 0;
    for (int p = p0 + lane; p - lane < p1; p += 64) {
        const bool live = p < p1;
        const int my = e;
        if (p + 64 < p1) e = g.idx[p + 64];
        uint64_t same = __ballot(live);           // live lanes with this lane's expert
        for (int bit = 1; bit < g.n; bit <<= 1) {
            const uint64_t b = __ballot(my & bit);
            same &= my & bit ? b : ~b;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1));
        if (live) {
            const int w = next[wv][my] + rank;
            g.tok[w] = p / g.k;
            g.pos[p] = w;
        }
        wave_sync();                              // every lane has read before the count moves on
        if (live && rank == 0) next[wv][my] += __popcll(same);
        wave_sync();                              // and reads the new one
    }
}

struct GemmArgs {
    const uint16_t *a;        // gate/up: X bf16 [T][d] (rows gathered by token); down: H bf16 [P][f]
    const uint8_t *pool;      // expert slabs
    uint64_t slab_stride;
    const int32_t *off;       // [n+1] first sorted pair of each expert
    const int32_t *toff;      // [n+1] first M tile of each expert
    const int32_t *tok;       // [P] token of each sorted pair
    const TilePlan *plan;     // [8] one per XCD
    int n, d, f;
    int ntiles;               // N tiles
    int slots;                // work groups per XCD
    int maxparts, prows;      // part buffers per XCD and their rows
    float *part;              // fp32 sums of the K parts, [8][maxparts][prows][kTileN]
    uint16_t *h;              // gate/up output, bf16 [P][f]
    float *y;                 // down output, fp32 [planes][P][d]
    int planes;
    size_t plane;             // P d
};

// Grouped GEMM, 8 waves per work group, one work group per CU, looping over its tiles.
//
// A tile is up to 256 tokens of one expert by 256 weight rows (gate/up: 128 W1 rows and the
// same 128 W3 rows). Two waves split the tokens and four the weight rows: a wave owns
// 16 HB tokens and 64 weight rows (gate/up: 32 W1 rows and the matching W3 rows, so an
// output's gate and up values sit in the same lane), so a token operand read from LDS serves
// 4 MFMAs and a weight operand HB. Both operands go from memory to LDS with direct loads (16 bytes per lane,
// the 128 bytes of a K step of 8 rows per instruction), in rings of stages of one K step
// each; one barrier per step. The token ring is shorter than the weight ring where LDS is
// short: it is refilled from the L2 and the weights from HBM. In a stage, row r's 16-byte
// chunk c sits at slot c ^ (r mod 8), which the loads arrange by permuting the source
// addresses within a row, so that the operand reads (16 rows, one chunk each per quarter
// wave) touch all banks evenly (no bank conflict counted).
//
// The weights are the MFMA's A operand, so a lane's four results are consecutive output
// columns of one token.
//
// Measured (us per layer, before: 192-token tiles, weights through registers, 4 fp32
// partial planes of the down projection; SiLU the same): 512 tokens on 8 Mixtral-shaped
// experts 613 -> 538, 4096 tokens 4106 -> 2580 (matrix cores busy 60 % of the cycles, at
// 1.9 GHz), 1333 tokens on 64 fine-grained experts 1285 -> 832. At 512 tokens the K loop
// takes as long with its MFMAs and operand reads removed: the load stream bounds it. Rings
// of 32-wide stages (deeper, 64-byte row pieces), waves that only load tokens or only
// weights, and raised wave priority around the MFMAs were no faster.
//
// A whole down tile sums all of f in one fp32 accumulator per output, where four parts of f
// were added before. With h exact the sums alone are then 5.0e-7 off (2-norm, against 64 bits)
// for f = 14336 instead of 2.0e-7, and 1.5e-7 instead of 1.0e-7 for f = 2560; split tiles are
// as before or closer. The bf16 rounding of x and h puts the outputs 2.9e-3 off either way.
constexpr int kRowBytes = kBK * 2;
constexpr int kRows = 1024 / kRowBytes;             // rows per load instruction of a wave
constexpr int kBBytes = kTileN * kRowBytes;         // weight rows of a stage
constexpr int kBLoads = kTileN / kRows / 8;         // load instructions per wave and stage
typedef __attribute__((address_space(1))) const void global_cvoid;
typedef __attribute__((address_space(3))) void lds_void;

template <int HB>
struct TileCfg {
    static constexpr int kABytes = HB * 32 * kRowBytes;           // token rows of a stage
    static constexpr int kAStages = HB <= 2 ? 4 : HB <= 5 ? 3 : 2;
    static constexpr int kBStages = HB <= 2 ? 4 : 3;
    static constexpr int kBBase = kAStages * kABytes;             // the weight ring follows the token ring
    static constexpr int kALoads = (HB + 1) / 2;                  // load instructions per wave and stage
    static constexpr int kLoads = kALoads + kBLoads;
    static constexpr int kRing = HB == 8 || HB == 6 || HB == 4 ? 4 : HB;   // divides 2 HB
    static constexpr int kAhead = kRing < 4 ? kRing : 4;
    // at a hand-over, loads that may be outstanding: those of stages after the next one
    static constexpr int kKeep = kAStages == kBStages ? (kAStages - 2) * kLoads : kBLoads;
    static_assert(kBBase + kBStages * kBBytes <= kLdsBytes, "the rings fit LDS");
    static_assert(kAStages == kBStages || (kAStages == 2 && kBStages == 3), "kKeep");
};

// The LDS reads of the previous step are done and at most N of this wave's loads are still
// in flight; then every wave of the work group is at this point.
template <int N>
__device__ __forceinline__ void wait_and_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
template <bool kGateUp, bool kOnce, int HB>
__device__ __forceinline__ void gemm_tile(const GemmArgs &g, uint8_t *lds, int e, int row0, int rows, int nt, int k0,
                                          int nsteps, int start, float *part, float *y)
{
    using C = TileCfg<HB>;
    constexpr int NA = C::kAStages, NB = C::kBStages, P = C::kAhead, R = C::kRing, kItems = 2 * HB;
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));   // keeps the addresses of all tile heights from being computed up front
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv & 1, wn = wv >> 1;
    const int K = kGateUp ? g.d : g.f;
    // row within a load instruction and byte offset of the chunk that lands in this lane's slot
    const int lr = lane >> 3, lc = ((lane & 7) ^ lr) * 16;

    // Token rows: loads past the stage's last repeat it, rows past the tile read its first.
    const uint8_t *asrc[C::kALoads];
    const uint8_t *const abase = reinterpret_cast<const uint8_t *>(g.a + (size_t)k0 * kBK);
#pragma unroll
    for (int j = 0; j < C::kALoads; ++j) {
        int r = min(j * 8 + wv, HB * 4 - 1) * kRows + lr;
        r = r < rows ? r : 0;
        asrc[j] = abase + operand_offset(kGateUp ? g.tok[row0 + r] : row0 + r, K, lc);
    }
    // Weight rows: instruction i of wave wv reads the kRows rows from 64 i + 8 wv; gate/up's
    // second half are the W3 rows, and a down tile with only 128 rows left in W2 (d an odd
    // multiple of 128) reads them twice.
    const size_t wrow = (size_t)nt * (kGateUp ? kGuCols : kTileN) + wv * kRows;
    const uint8_t *const bbase = g.pool + (uint64_t)e * g.slab_stride +
                                 2 * ((kGateUp ? (size_t)0 : (size_t)2 * g.f * g.d) + wrow * K + (size_t)k0 * kBK);
    const size_t bhalf = kGateUp ? (size_t)2 * g.f * K : nt * kTileN + 128 < g.d ? (size_t)256 * K : 0;
    const size_t bquarter = operand_offset(64, K, 0);
    const size_t blane = operand_offset(lr, K, lc);
    auto koff = [&](int stage) {   // steps go round from `start`
        const int ks = stage + start;
        return (size_t)(ks >= nsteps ? ks - nsteps : ks) * kRowBytes;
    };
    auto load_a = [&](int i, int stage, int buf) {
        __builtin_amdgcn_global_load_lds((global_cvoid *)(asrc[i] + koff(stage)),
                                         (lds_void *)(lds + buf * C::kABytes + min(i * 8 + wv, HB * 4 - 1) * 1024), 16, 0,
                                         0);
    };
    auto load_b = [&](int i, int stage, int buf) {
        const uint8_t *src = bbase + koff(stage) + (i >> 1) * bhalf + (i & 1) * bquarter;
        __builtin_amdgcn_global_load_lds((global_cvoid *)(src + blane),
                                         (lds_void *)(lds + C::kBBase + buf * kBBytes + (i * 8 + wv) * 1024), 16, 0,
                                         kOnce ? 2 : 0);   // 2: nontemporal
    };

    floatx4_t acc[HB][4];
#pragma unroll
    for (int m = 0; m < HB; ++m)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[m][nb] = floatx4_t{0.f, 0.f, 0.f, 0.f};

    // Operand reads: row lane % 16 of a block, chunk 4 kb + lane / 16. The items of a step are
    // (kb, m) in order; item j's token block is read P items before its MFMAs, in a ring of R
    // registers, and the weight blocks of a kb with its first item. P items before the end
    // of a step its reads are all issued: there the wave waits for them and for the next
    // step's loads, and after the barrier the buffers just read take the loads of the steps
    // NA (tokens) and NB (weights) after it, spread over the last P items.
    const int rd = (lane & 15) * kRowBytes + ((lane >> 4) ^ (lane & 7)) * 16;
    const uint8_t *const ra = lds + wm * HB * 16 * kRowBytes;
    const uint8_t *const rb = lds + C::kBBase + wn * (kGateUp ? 32 : 64) * kRowBytes;
    bf16x8_t wf[2][4], tf[R];
    auto read_item = [&](int j, int ba, int bb) {
        const int kb = j / HB, sl = rd ^ (kb * 64);
        if (j % HB == 0) {
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const int o = kGateUp ? (nb >> 1) * kGuCols + (nb & 1) * 16 : nb * 16;
                wf[kb][nb] = *reinterpret_cast<const bf16x8_t *>(rb + bb * kBBytes + o * kRowBytes + sl);
            }
        }
        tf[j % R] = *reinterpret_cast<const bf16x8_t *>(ra + ba * C::kABytes + (j % HB) * 16 * kRowBytes + sl);
    };
    auto mma = [&](int j, const bf16x8_t t) {
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
            acc[j % HB][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j / HB][nb], t, acc[j % HB][nb], 0, 0, 0);
    };
#pragma unroll
    for (int q = 0; q < NB; ++q) {
        if (q >= nsteps) continue;
        if (q < NA)
#pragma unroll
            for (int i = 0; i < C::kALoads; ++i) load_a(i, q, q);
#pragma unroll
        for (int i = 0; i < kBLoads; ++i) load_b(i, q, q);
    }
    if (nsteps >= NB) wait_and_barrier<(NA - 1) * C::kALoads + (NB - 1) * kBLoads>();
    else wait_and_barrier<0>();
#pragma unroll
    for (int j = 0; j < P; ++j) read_item(j, 0, 0);
    int s = 0, ba = 0, bb = 0;
    // One step. Steps that still have all loads to issue have no branch in them.
    enum { kSteady, kDrain, kFinal };
    auto step = [&](auto mode) {
        constexpr bool kLast = decltype(mode)::value == kFinal, kFull = decltype(mode)::value == kSteady;
        const int na = ba + 1 == NA ? 0 : ba + 1, nb = bb + 1 == NB ? 0 : bb + 1;
#pragma unroll
        for (int j = 0; j < kItems; ++j) {
            const int at = j - (kItems - P);   // items since the hand-over
            if (at == 0 && !kLast) {
                if (kFull || s + NB - 1 < nsteps) wait_and_barrier<C::kKeep>();
                else wait_and_barrier<0>();
            }
            if (at >= 0 && !kLast) {
                constexpr int kEach = (C::kLoads + P - 1) / P;
#pragma unroll
                for (int i = at * kEach; i < (at + 1) * kEach && i < C::kLoads; ++i) {
                    if (i < C::kALoads) {
                        if (kFull || s + NA < nsteps) load_a(i, s + NA, ba);
                    } else if (kFull || s + NB < nsteps) {
                        load_b(i - C::kALoads, s + NB, bb);
                    }
                }
            }
            const bf16x8_t t = tf[j % R];
            if (at < 0) read_item(j + P, ba, bb);
            else if (!kLast) read_item(j + P - kItems, na, nb);
            mma(j, t);
            __builtin_amdgcn_sched_barrier(0);
        }
        ++s;
        ba = na;
        bb = nb;
    };
    while (s + NB < nsteps) step(std::integral_constant<int, kSteady>{});
    while (s + 1 < nsteps) step(std::integral_constant<int, kDrain>{});
    step(std::integral_constant<int, kFinal>{});

    // result r of a 16x16 block: weight row 4 (lane / 16) + r, token lane % 16
    const int c4 = 4 * (lane >> 4);
#pragma unroll
    for (int m = 0; m < HB; ++m) {
        const int tr = (wm * HB + m) * 16 + (lane & 15);
        if (tr >= rows) continue;
        if (part) {
            float *dst = part + (size_t)tr * kTileN + c4;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) {
                const int col = kGateUp ? (nb >> 1) * kGuCols + wn * 32 + (nb & 1) * 16 : wn * 64 + nb * 16;
                *reinterpret_cast<floatx4_t *>(dst + col) = acc[m][nb];
            }
        } else if constexpr (kGateUp) {
            uint16_t *dst = g.h + (size_t)(row0 + tr) * g.f + nt * kGuCols + wn * 32 + c4;
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                const floatx4_t gv = acc[m][nb], uv = acc[m][nb + 2];
                uint2 o;
                o.x = swiglu_bf(gv[0], uv[0]) | ((uint32_t)swiglu_bf(gv[1], uv[1]) << 16);
                o.y = swiglu_bf(gv[2], uv[2]) | ((uint32_t)swiglu_bf(gv[3], uv[3]) << 16);
                *reinterpret_cast<uint2 *>(dst + nb * 16) = o;
            }
        } else {
            const int col0 = nt * kTileN + wn * 64 + c4;
            float *dst = y + (size_t)(row0 + tr) * g.d + col0;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                if (col0 + nb * 16 < g.d) *reinterpret_cast<floatx4_t *>(dst + nb * 16) = acc[m][nb];
        }
    }
}

// kOnce: the weights are read about once (nontemporal loads).
template <bool kGateUp, bool kOnce>
__global__ __launch_bounds__(kGemmThreads) void k_moe_gemm(GemmArgs g)
{
    __shared__ __align__(1024) uint8_t lds[kLdsBytes];
    const int lane = threadIdx.x & 63;
    const int xcd = blockIdx.x % kXcds;
    const TilePlan p = g.plan[xcd];
    const int nunits = p.full + (p.units - p.full) * p.s;
    const int nsteps = (kGateUp ? g.d : g.f) / kBK;
    int tbase[MOE_MAX_EXPERTS / 64];   // first tile of experts lane, lane + 64, ...
#pragma unroll
    for (int i = 0; i < MOE_MAX_EXPERTS / 64; ++i) {
        const int e = lane + 64 * i;
        tbase[i] = e < g.n ? g.toff[e] * g.ntiles : 0x7fffffff;
    }
    for (int u = blockIdx.x / kXcds; u < nunits; u += g.slots) {
        int t = u, ks = 0, parts = 1;
        float *part = nullptr, *y = g.y;
        if (u >= p.full) {
            const int v = u - p.full;
            t = p.full + v / p.s;
            ks = v % p.s;
            parts = p.s;
            if (!kGateUp && p.s <= g.planes) y += ks * g.plane;
            else part = g.part + ((size_t)xcd * g.maxparts + v) * g.prows * kTileN;
        }
        t += p.u0;
        int e = -1;   // the last expert whose first tile is at or before t
#pragma unroll
        for (int i = 0; i < MOE_MAX_EXPERTS / 64; ++i) e += __popcll(__ballot(tbase[i] <= t));
        const int o0 = g.off[e], c = g.off[e + 1] - o0;
        t -= g.toff[e] * g.ntiles;
        const int m = tiles_of(c), mt = t % m, nt = t / m;
        const int r0 = tile_row(c, mt), row0 = o0 + r0, rows = tile_row(c, mt + 1) - r0;
        const int k0 = nsteps * ks / parts, kn = nsteps * (ks + 1) / parts - k0;
        // An expert's N tiles run side by side. With one M tile each walks its weights from a
        // start of its own, so that they read different columns at a time (neighbours 256
        // bytes apart: Mixtral-shaped 512-token layer 570 -> 527 us, 7 steps apart 538); with
        // more, the tiles that share weights or tokens stay in step for the L2.
        const int start = m == 1 ? (int)((unsigned)(nt * kStagger) % (unsigned)kn) : 0;
        switch ((rows + 31) >> 5) {
#define MOE_HB_CASE(N) \
    case N: gemm_tile<kGateUp, kOnce, N>(g, lds, e, row0, rows, nt, k0, kn, start, part, y); break;
            MOE_HB_CASE(1) MOE_HB_CASE(2) MOE_HB_CASE(3) MOE_HB_CASE(4)
            MOE_HB_CASE(5) MOE_HB_CASE(6) MOE_HB_CASE(7) MOE_HB_CASE(8)
#undef MOE_HB_CASE
        default: break;
        }
        wait_and_barrier<0>();   // the last stage is read before the next tile's loads overwrite it
    }
}

// H of the gate/up tiles split over K: h = SiLU(sum of the g parts) * (sum of the u parts),
// the parts added in order. Work group b: XCD b mod 8, then split tile i of that XCD and a
// block of 16 of its rows; each thread takes 4 consecutive columns of 2 rows.
constexpr int kTailRows = 16;
__global__ __launch_bounds__(kThreads) void k_tail_combine(GemmArgs g)
{
    constexpr int kQuads = kGuCols / 4;  // 4-column groups of the tile's columns
    const int xcd = blockIdx.x % kXcds;
    const int i = (blockIdx.x / kXcds) % g.slots;
    const int rb = blockIdx.x / kXcds / g.slots;
    const TilePlan p = g.plan[xcd];
    if (i >= p.units - p.full) return;
    int t = p.u0 + p.full + i;
    int lo = 0, hi = g.n - 1;   // the last expert whose first tile is at or before t
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (g.toff[mid] * g.ntiles <= t) lo = mid;
        else hi = mid - 1;
    }
    const int o0 = g.off[lo], c0 = g.off[lo + 1] - o0;
    t -= g.toff[lo] * g.ntiles;
    const int m = tiles_of(c0), mt = t % m, nt = t / m;
    const int r0 = tile_row(c0, mt), row0 = o0 + r0, rows = tile_row(c0, mt + 1) - r0;
    const float *p0 = g.part + ((size_t)xcd * g.maxparts + (size_t)i * p.s) * g.prows * kTileN;
    for (int c = threadIdx.x; c < kTailRows * kQuads; c += kThreads) {
        const int tr = rb * kTailRows + c / kQuads, col = (c % kQuads) * 4;
        if (tr >= rows) continue;
        float4 gv = make_float4(0.f, 0.f, 0.f, 0.f), uv = gv;
        for (int j = 0; j < p.s; ++j) {
            const float *pj = p0 + ((size_t)j * g.prows + tr) * kTileN + col;
            const float4 a = *reinterpret_cast<const float4 *>(pj);
            const float4 b = *reinterpret_cast<const float4 *>(pj + kGuCols);
            gv.x += a.x; gv.y += a.y; gv.z += a.z; gv.w += a.w;
            uv.x += b.x; uv.y += b.y; uv.z += b.z; uv.w += b.w;
        }
        uint2 o;
        o.x = swiglu_bf(gv.x, uv.x) | ((uint32_t)swiglu_bf(gv.y, uv.y) << 16);
        o.y = swiglu_bf(gv.z, uv.z) | ((uint32_t)swiglu_bf(gv.w, uv.w) << 16);
        *reinterpret_cast<uint2 *>(g.h + (size_t)(row0 + tr) * g.f + nt * kGuCols + col) = o;
    }
}

// OUT[t][i] = sum_r w[t][r] * y of pair (t, r), four consecutive i per thread. The y of a
// tile split over K is the sum of its parts, in order; of any other tile, the GEMM's output.
// Work group b covers token b / nparts, columns (b mod nparts) * 1024 ...
__global__ __launch_bounds__(kThreads) void k_prefill_combine(GemmArgs g, const int32_t *idx, const int32_t *pos,
                                                              const float *w, int k, int nparts, float *out)
{
    const int t = blockIdx.x / nparts;
    const int i = ((blockIdx.x % nparts) * kThreads + threadIdx.x) * 4;
    if (i >= g.d) return;
    const int U = g.toff[g.n] * g.ntiles;
    const int nt = i / kTileN;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int r = 0; r < k; ++r) {
        const int e = idx[t * k + r], pr = pos[t * k + r];
        const int o0 = g.off[e], c = g.off[e + 1] - o0;
        const int mt = tile_of_row(c, pr - o0);
        const int u = g.toff[e] * g.ntiles + nt * tiles_of(c) + mt;
        const int xcd = xcd_of_tile(U, u);
        const TilePlan p = g.plan[xcd];
        const int v = u - p.u0 - p.full;
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        if (v < 0 || p.s <= g.planes) {
            const float *src = g.y + (size_t)pr * g.d + i;
            s = *reinterpret_cast<const float4 *>(src);
            for (int q = 1; v >= 0 && q < p.s; ++q) {
                const float4 a = *reinterpret_cast<const float4 *>(src + q * g.plane);
                s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w;
            }
        } else {
            const float *src = g.part + (((size_t)xcd * g.maxparts + (size_t)v * p.s) * g.prows + (pr - o0 - tile_row(c, mt))) *
                                            kTileN + i % kTileN;
            for (int q = 0; q < p.s; ++q) {
                const float4 a = *reinterpret_cast<const float4 *>(src + (size_t)q * g.prows * kTileN);
                s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w;
            }
        }
        const float wr = w[t * k + r];
        acc.x = fmaf(wr, s.x, acc.x);
        acc.y = fmaf(wr, s.y, acc.y);
        acc.z = fmaf(wr, s.z, acc.z);
        acc.w = fmaf(wr, s.w, acc.w);
    }
    *reinterpret_cast<float4 *>(out + (size_t)t * g.d + i) = acc;
}

constexpr size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

struct PrefillWs {
    uint16_t *xb;
    int32_t *idx, *off, *tok, *pos, *toff;
    float *w;
    uint16_t *h;
    TilePlan *plan;
    float *y;
    float *gu_part, *dn_part;   // gate/up part buffers (y is written later), down part buffers
    int gu_parts, dn_parts;     // their number per XCD
    int planes;                 // of y
};

// Rows of a part buffer: an expert has at most T tokens.
int part_rows(int T) { return std::min(T, kTileM); }

// The workspace with that many planes of y; its size is returned.
size_t layout(int d, int f, int n, int k, int T, int nplanes, uint8_t *base, PrefillWs *ws)
{
    const size_t P = (size_t)T * k;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align256(bytes);
        return base ? base + at : nullptr;
    };
    uint8_t *xb = take((size_t)T * d * 2);
    uint8_t *idx = take(P * 4);
    uint8_t *w = take(P * 4);
    uint8_t *off = take((size_t)(n + 1) * 4);
    uint8_t *tok = take(P * 4);
    uint8_t *pos = take(P * 4);
    uint8_t *h = take(P * f * 2);
    uint8_t *toff = take((size_t)(n + 1) * 4);
    uint8_t *plan = take(sizeof(TilePlan) * 2 * kXcds);
    // fp32 sums: the planes of y, which also hold gate/up's part buffers before y is written,
    // and from 64 tokens per expert on, where a part buffer has many rows, 48 MiB more for the
    // part buffers of both; fewer part buffers only mean fewer K splits
    const size_t planes = (size_t)nplanes * P * d * 4;
    const size_t extra = (int64_t)T * k < (int64_t)64 * n ? 0 : (size_t)48 << 20;
    uint8_t *y = take(planes);
    uint8_t *parts = take(extra);
    if (ws) {
        ws->xb = reinterpret_cast<uint16_t *>(xb);
        ws->idx = reinterpret_cast<int32_t *>(idx);
        ws->w = reinterpret_cast<float *>(w);
        ws->off = reinterpret_cast<int32_t *>(off);
        ws->tok = reinterpret_cast<int32_t *>(tok);
        ws->pos = reinterpret_cast<int32_t *>(pos);
        ws->h = reinterpret_cast<uint16_t *>(h);
        ws->toff = reinterpret_cast<int32_t *>(toff);
        ws->plan = reinterpret_cast<TilePlan *>(plan);
        const size_t set = (size_t)kXcds * part_rows(T) * kTileN * 4;   // one buffer on every XCD
        ws->y = reinterpret_cast<float *>(y);
        ws->planes = nplanes;
        ws->gu_part = ws->y;
        // none below 16 tokens: such a layer is short, its memory holds few part buffers, and
        // the launch that adds them takes 5 us (which is also why they are not more where y
        // has more than four planes: 64 tokens on 8 experts of d = 1152, f = 2048 41.8 against
        // 42.8 us)
        const size_t gu = (size_t)std::min(nplanes, 4) * P * d * 4 + extra;
        ws->gu_parts = T < 16 ? 0 : (int)std::min<size_t>(kMaxParts, gu / set);
        ws->dn_part = reinterpret_cast<float *>(parts);
        ws->dn_parts = (int)std::min<size_t>(kMaxParts, extra / set);
    }
    return o;
}

}  // namespace

size_t prefill_workspace_bytes(int d, int f, int n, int k, int T)
{
    return layout(d, f, n, k, T, max_planes(T), nullptr, nullptr);
}

// The least that is taken is what was recommended before the tile tables were kept in the
// workspace: four planes without the room for the tables, which then hold fewer. One plane and
// the tables always fit it: three planes are 3 T k d values, at least 3 * 128.
constexpr size_t table_bytes(int n) { return align256((size_t)(n + 1) * 4) + align256(sizeof(TilePlan) * 2 * kXcds); }
static_assert(table_bytes(MOE_MAX_EXPERTS) <= (size_t)3 * 128 * 4, "one plane and the tables fit the least workspace");

size_t prefill_workspace_min(int d, int f, int n, int k, int T)
{
    return layout(d, f, n, k, T, 4, nullptr, nullptr) - table_bytes(n);
}

hipError_t launch_prefill(const PrefillPlan &P, const float *X, float *OUT, int32_t *idx, float *w, void *wsp,
                          size_t ws_bytes, hipStream_t s)
{
    PrefillWs ws{};
    int planes = max_planes(P.T);
    while (planes > 1 && layout(P.d, P.f, P.n, P.k, P.T, planes, nullptr, nullptr) > ws_bytes) --planes;
    if (layout(P.d, P.f, P.n, P.k, P.T, planes, static_cast<uint8_t *>(wsp), &ws) > ws_bytes) return hipErrorInvalidValue;
    int32_t *idx_d = idx ? idx : ws.idx;
    float *w_d = w ? w : ws.w;
    hipError_t e;
    if ((e = launch_router(X, P.wr, P.T, P.d, P.n, P.k, idx_d, w_d, s)) != hipSuccess) return e;
    const int slots = std::max(1, device_cu_count() / kXcds);

    GroupArgs ga{};
    ga.idx = idx_d;
    ga.npairs = P.T * P.k;
    ga.n = P.n;
    ga.k = P.k;
    ga.off = ws.off;
    ga.toff = ws.toff;
    ga.tok = ws.tok;
    ga.pos = ws.pos;
    ga.plan = ws.plan;
    ga.ntiles[0] = P.f / kGuCols;
    ga.ntiles[1] = (P.d + kTileN - 1) / kTileN;
    ga.nsteps[0] = P.d / kBK;
    ga.nsteps[1] = P.f / kBK;
    ga.maxparts[0] = ws.gu_parts;
    ga.maxparts[1] = ws.dn_parts;
    ga.slots = slots;
    ga.planes = ws.planes;
    ga.x = X;
    ga.xb = ws.xb;
    ga.n8 = (int64_t)P.T * P.d / 8;
    const int cast_blocks = (int)std::min<int64_t>((ga.n8 + kGroupThreads - 1) / kGroupThreads, 1024);
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_group, dim3(1 + cast_blocks), dim3(kGroupThreads), 0, s, ga);
    if ((e = hipGetLastError()) != hipSuccess) return e;

    GemmArgs g{};
    g.pool = P.pool;
    g.slab_stride = P.slab_stride;
    g.off = ws.off;
    g.toff = ws.toff;
    g.tok = ws.tok;
    g.n = P.n;
    g.d = P.d;
    g.f = P.f;
    g.slots = slots;
    g.prows = part_rows(P.T);
    g.h = ws.h;
    g.y = ws.y;
    g.planes = ws.planes;
    g.plane = (size_t)P.T * P.k * P.d;

    g.a = ws.xb;
    g.plan = ws.plan;
    g.ntiles = ga.ntiles[0];
    g.maxparts = ws.gu_parts;
    g.part = ws.gu_part;
    // Below one full M tile per expert on average the weights go by once and are loaded
    // nontemporally (Mixtral-shaped 512 tokens: 578 -> 527 us, Phi 27 tokens: 439 -> 390 us);
    // from there on M tiles share them through the caches (4096 tokens: 2516 us, nontemporal
    // 2590 us; 1024 tokens, 256 per expert: 928 and 960 us).
    const bool once = (int64_t)P.T * P.k < (int64_t)kTileM * P.n;
    const dim3 grid(kXcds * slots), block(kGemmThreads);
    if (once) hipLaunchKernelGGL((k_moe_gemm<true, true>), grid, block, 0, s, g);
    else hipLaunchKernelGGL((k_moe_gemm<true, false>), grid, block, 0, s, g);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (g.maxparts > 1) {
        const int row_blocks = (g.prows + kTailRows - 1) / kTailRows;
        hipLaunchKernelGGL(k_tail_combine, dim3(kXcds * slots * row_blocks), dim3(kThreads), 0, s, g);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }

    g.a = ws.h;
    g.plan = ws.plan + kXcds;
    g.ntiles = ga.ntiles[1];
    g.maxparts = ws.dn_parts;
    g.part = ws.dn_part;
    if (once) hipLaunchKernelGGL((k_moe_gemm<false, true>), grid, block, 0, s, g);
    else hipLaunchKernelGGL((k_moe_gemm<false, false>), grid, block, 0, s, g);
    if ((e = hipGetLastError()) != hipSuccess) return e;

    const int nparts = (P.d + 4 * kThreads - 1) / (4 * kThreads);
    hipLaunchKernelGGL(k_prefill_combine, dim3(P.T * nparts), dim3(kThreads), 0, s, g, idx_d, ws.pos, w_d, P.k, nparts,
                       OUT);
    return hipGetLastError();
}

}  // namespace moe

extern "C" {

size_t moe_prefill_workspace_bytes(const moe_prefill_desc *P, int T)
{
    if (!P || T < 0 || P->d <= 0 || P->f <= 0 || P->n <= 0 || P->k <= 0) return 0;
    return moe::prefill_workspace_bytes(P->d, P->f, P->n, P->k, T);
}

int moe_prefill_forward(const moe_prefill_desc *P, const float *X_dev, int T, float *OUT_dev, int32_t *idx_dev,
                        float *w_dev, void *workspace, size_t workspace_bytes, void *stream)
{
    MOE_GUARD_BEGIN
    MOE_REQUIRE(P, "moe_prefill_forward: null descriptor");
    MOE_REQUIRE(T >= 0, "moe_prefill_forward: T=%d < 0", T);
    MOE_REQUIRE(P->d > 0 && P->d % 128 == 0 && P->d <= MOE_MAX_D,
                "moe_prefill_forward: d=%d must be a multiple of 128 in [128,%d]", P->d, MOE_MAX_D);
    MOE_REQUIRE(P->f > 0 && P->f % 128 == 0, "moe_prefill_forward: f=%d must be a positive multiple of 128", P->f);
    MOE_REQUIRE(P->n >= 1 && P->n <= MOE_MAX_EXPERTS, "moe_prefill_forward: n=%d out of range", P->n);
    MOE_REQUIRE(P->k >= 1 && P->k <= P->n && P->k <= MOE_MAX_TOPK, "moe_prefill_forward: k=%d out of range", P->k);
    if (T == 0) return MOE_OK;
    MOE_REQUIRE(X_dev && OUT_dev && workspace && P->w_router && P->expert_pool, "moe_prefill_forward: null pointer");
    MOE_REQUIRE(moe::aligned16(X_dev) && moe::aligned16(OUT_dev) && moe::aligned16(P->w_router) &&
                    moe::aligned16(P->expert_pool),
                "moe_prefill_forward: device pointers must be 16-byte aligned");
    MOE_REQUIRE(((uintptr_t)workspace & 255u) == 0, "moe_prefill_forward: workspace not 256-byte aligned");
    const size_t need = moe::prefill_workspace_min(P->d, P->f, P->n, P->k, T);
    MOE_REQUIRE(workspace_bytes >= need, "moe_prefill_forward: workspace %zu < %zu bytes", workspace_bytes, need);
    moe::PrefillPlan plan{};
    plan.d = P->d;
    plan.f = P->f;
    plan.n = P->n;
    plan.k = P->k;
    plan.T = T;
    plan.wr = P->w_router;
    plan.pool = static_cast<const uint8_t *>(P->expert_pool);
    plan.slab_stride = moe_slab_bytes(P->d, P->f);
    MOE_HIP(moe::launch_prefill(plan, X_dev, OUT_dev, idx_dev, w_dev, workspace, workspace_bytes,
                                (hipStream_t)stream));
    return MOE_OK;
    MOE_GUARD_END
}

}  // extern "C"
