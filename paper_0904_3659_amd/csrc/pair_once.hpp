// The pair-once block evaluation of Eq. (gravity) (Sec. I), shared by the
// single-system forward kernel (forward_sym.hip) and the batched ensemble
// kernel (batched.hip).
//
// Every unordered pair is computed once: the term of pair (i, j) gives
// m_j d r^3 to a_i and, by the antisymmetry of the softened force (one eps2
// for all pairs), -m_i d r^3 to a_j; the potential term gives m_j r to p_i
// and m_i r to p_j.  That shares the difference, distance, rsqrt and r^3 of
// both ordered pairs.
//
// Blocks and the ring
//   A system of n particles is cut into M blocks of P = W*64*K.  The caller
//   (one workgroup) owns block I, chunk c of C: it keeps block I in VGPRs
//   (K rows per lane, W waves) and meets
//     - its own block (the diagonal), pair-once between different 64-row
//       tiles and as ordered pairs (j == i removed by index) within a tile,
//       and
//     - the blocks J = I + delta (mod M) for delta = 1..H_I (the ring), with
//       H_I = (M-1)/2, plus delta = M/2 when M is even and I < M/2,
//   so every unordered pair of distinct blocks is met exactly once.  The
//   block's tile sequence (diagonal tiles, then ring tiles delta-major) is
//   cut into the C chunks (chunk_begin; one_tile_plan).
//
// j-tiles of 64 particles are staged in LDS twice over (entries e and
// e + 64 hold particle e).  On a ring tile, lane l at step s (0..63) meets
// particle (l + s) mod 64 of the tile, read from entry l + s: each step is a
// permutation of the 64 particles over the 64 lanes, and the entry index
// needs no wrap, so the unrolled loop addresses LDS with immediate offsets
// from one base.  The j-side sums live in 128 per-wave LDS slots in the same
// way: at step s lane l adds its K terms to slot l + s (read-modify-write),
// so particle e collects in slots e and e + 64.  No two lanes touch the
// same slot in a step; a slot's next writer is another lane of the same
// wave, and one wave's LDS accesses complete in issue order, so the sums are
// exact read-modify-writes in a fixed order (no atomics; LDS atomics
// serialise and were 4x slower).  After the 64 steps the W waves' slot
// pairs are added in wave order and written as the tile's partial.
//
// Ring groups and partials.  The ring offsets are processed in groups of
// consecutive deltas, one launch per group, so that library memory stays
// O((C + G) n) instead of O(n^2 / P): launch g covers deltas [d_lo, d_hi)
// (the first group also the diagonal, delta 0) and writes float4 partials
// [C + G][n]: slots 0..C-1 hold the i-side sums of the C chunks over the
// group's tiles, slot C + delta - max(d_lo, 1) holds what particle j in
// block J received from block J - delta.  A fold kernel then adds each
// particle's slots of the group, in fixed order and in float64, to its
// running sum (the last group's fold rounds it and stores a, p).  No
// atomics, no cross-workgroup races: the result is bitwise reproducible for
// a given variant, n, chunk count and group size.
//
// Padding: rows past n take position +1e18 and mass 0, tile slots past n
// take -1e18 and mass 0, so padded terms are exactly zero for finite
// positions below 1e17 in magnitude.
#pragma once

#include "common.hpp"

#include <cstdlib>

namespace nbody {

constexpr float kPadRow = 1e18f;
constexpr float kPadCol = -1e18f;

// LDS entries per staged j-tile (64 particles, stored twice) and per wave's
// j-side slots.
constexpr int kTileLds = 128;
constexpr int kSlotLds = 128;

__host__ __device__ __forceinline__ int ring_len(int I, int M)
{
    return (M - 1) / 2 + (((M & 1) == 0 && I < M / 2) ? 1 : 0);
}

// Number of j-side slots block J of an M-block system receives.
__host__ __device__ __forceinline__ int ring_in(int J, int M)
{
    return (M - 1) / 2 + (((M & 1) == 0 && J >= M / 2) ? 1 : 0);
}

// The deltas of group [d_lo, d_hi) that have a j-side slot (the diagonal,
// delta 0, has none): [max(d_lo, 1), d_hi).
__host__ __device__ __forceinline__ int group_first_delta(int d_lo) { return d_lo > 0 ? d_lo : 1; }

// Fold of one ring group: particle j (block J) adds its C chunk slots and
// the j-side slots of the group's deltas its block received, deltas
// [dj, min(d_hi, ring_in(J, M) + 1)), in slot order, each widened to
// float64.  Four groups of 64 threads each add a contiguous quarter of the
// slots, and the four group sums are added in group order; the group's sum
// is then added to the particle's running sum acc (FIRST: acc is not read;
// LAST: the result is rounded once and xyz goes to out3[j][3], w to out1[j],
// skipped when out1 is NULL, followed by the leap-frog update `e` with EPI).
// A fixed order throughout: bitwise reproducible.  A workgroup covers 64
// particles.  acc is [n] double4 and is neither read nor written when the
// fold is both FIRST and LAST.
template <int PB, bool EPI = false>
__global__ __launch_bounds__(256) void slot_fold_kernel(const float4 *__restrict__ partial, int n,
                                                        int M, int C, int d_lo, int d_hi,
                                                        int first, int last, double4 *acc,
                                                        float *out3, float *out1, LfEpi e)
{
    __shared__ double4 red[4][64];
    const int l = threadIdx.x & 63;
    const int g = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + l;
    double4 s = make_double4(0.0, 0.0, 0.0, 0.0);
    if (j < n) {
        const int dj = group_first_delta(d_lo);
        const int recv = min(d_hi, ring_in(j / PB, M) + 1) - dj;
        const int S = C + (recv > 0 ? recv : 0);
        const int q = (S + 3) / 4;
        const int k1 = min(S, (g + 1) * q);
#pragma unroll 4
        for (int k = g * q; k < k1; ++k) {
            const float4 v = partial[(size_t)k * n + j];
            s.x += (double)v.x;
            s.y += (double)v.y;
            s.z += (double)v.z;
            s.w += (double)v.w;
        }
    }
    red[g][l] = s;
    __syncthreads();
    if (g != 0 || j >= n) return;
    double4 t = red[0][l];
#pragma unroll
    for (int g2 = 1; g2 < 4; ++g2) {
        const double4 v = red[g2][l];
        t.x += v.x;
        t.y += v.y;
        t.z += v.z;
        t.w += v.w;
    }
    if (!first) {
        const double4 r = acc[j];
        t.x += r.x;
        t.y += r.y;
        t.z += r.z;
        t.w += r.w;
    }
    if (!last) {
        acc[j] = t;
        return;
    }
    const float4 f = make_float4((float)t.x, (float)t.y, (float)t.z, (float)t.w);
    if constexpr (EPI) {
        lf_finish(e, j, f, out3, out1);
    } else {
        out3[3 * j + 0] = f.x;
        out3[3 * j + 1] = f.y;
        out3[3 * j + 2] = f.z;
        if (out1) out1[j] = f.w;
    }
}

// Launch plan of a single-system pair-once evaluation: M blocks of P
// particles, C chunks per block, D = M/2 ring deltas processed in `groups`
// launches of G deltas each (the first also the diagonal).  Workspace:
// partials [C + G][n] float4 and, with more than one group, a float64
// running sum [n] double4.
struct SymPlan {
    int M = 0, C = 0, G = 0, groups = 0;
    size_t partial_bytes = 0, acc_bytes = 0;
    size_t bytes() const { return partial_bytes + acc_bytes; }
};

// Plan for n particles in blocks of P, given the number of workgroups the
// device holds at once (resident; the chunk count fills them, divided by
// occ) and a workspace budget in bytes.  Returns false if even one delta
// per group and one chunk per block exceed the budget.
inline bool sym_plan(int64_t n, int P, int64_t resident, int occ, size_t budget, SymPlan *out)
{
    SymPlan pl;
    const int TPB = P / 64;
    pl.M = (int)((n + P - 1) / P);
    const int D = pl.M / 2;  // ring deltas 1..D
    int64_t C = resident / ((int64_t)pl.M * occ);
    const int64_t max_c = (int64_t)(D + 1) * TPB;  // tiles of a block's sequence
    C = C < 1 ? 1 : (C > max_c ? max_c : C);
    const size_t slot = 16 * (size_t)n;          // one float4 per particle
    const int64_t slots = (int64_t)(budget / slot);
    if (C + D <= slots || D == 0) {
        pl.C = (int)C;
        pl.G = D;
        pl.groups = 1;
    } else {
        // several groups: room for C + G slots plus the running sum (two
        // slots' worth); the chunks take at most half of the slots
        if (slots < 4) return false;
        const int64_t half = (slots - 2) / 2;
        if (C > half) C = half;
        const int64_t gmax = slots - C - 2;
        pl.groups = (int)((D + gmax - 1) / gmax);
        pl.G = (D + pl.groups - 1) / pl.groups;
        const int64_t cg = (int64_t)pl.G * TPB;  // tiles per block in a later group
        pl.C = (int)(C > cg ? cg : C);
    }
    // the running sum starts on a 256-byte boundary (double4 needs 32)
    pl.partial_bytes = (slot * (size_t)(pl.C + pl.G) + 255) / 256 * 256;
    pl.acc_bytes = pl.groups > 1 ? 32 * (size_t)n : 0;
    *out = pl;
    return true;
}

// Ring deltas [d_lo, d_hi) of group g of a plan (delta 0, the diagonal, is
// in group 0).
inline void sym_group(const SymPlan &pl, int g, int *d_lo, int *d_hi)
{
    *d_lo = g == 0 ? 0 : 1 + g * pl.G;
    const int hi = 1 + (g + 1) * pl.G;
    *d_hi = hi < pl.M / 2 + 1 ? hi : pl.M / 2 + 1;
}

// First tile of chunk c of the C chunks a block's U tiles are cut into (c == C:
// U).  Every chunk has one tile; the other U - C are dealt in equal shares to
// the first half of the chunks and in shares falling linearly to nothing over
// the second half, what is left of a tile to the later chunk (with fewer than two
// tiles to a chunk the last one may so be among the longer ones; up to the
// earlier chunk it took 0.7% longer at 65,536 bodies, level at 50,021 and from
// 100,000).  The grid runs chunk-major (all blocks' first chunks, then all second
// ones, ...), so a launch ends on its smaller workgroups instead of on equal
// ones; no chunk has more than 2 + 4/3 (U - C) / C tiles.  With C equal chunks of
// 1/8 of a slot's share, the last of eight rounds left CUs idle for 5-12% of the
// launch (65,536 and 2^18 bodies, 92 and 87% CU-busy).
__host__ __device__ __forceinline__ int chunk_begin(int U, int C, int c)
{
    if (U <= C) return c < U ? c : U;
    if (c == C) return U;
    const float x = (float)c / (float)C;
    const float t = fmaxf(x - 0.5f, 0.0f);
    return c + (int)((float)(U - C) * (4.0f / 3.0f) * (x - t * t));
}

// Tiles a chunk of a plan whose blocks hold TPB tiles may have (chunk_begin's bound,
// in the first group).
inline int longest_chunk(const SymPlan &pl, int TPB)
{
    const int U = (pl.G + 1) * TPB;
    return U <= pl.C ? 1 : 2 + (int)(4LL * (U - pl.C) / (3LL * pl.C));
}

// Tiles whose sums a row holds in float32 registers before they go to the chunk's
// partial: a float32 sum over every tile of a long chunk loses more than the rest
// of a row's sums together (from 64 tiles on; 2^18 bodies).  A hand-over reads and
// writes a partial per row (every 16 tiles wrote 12.3 GiB at 2^20 bodies, and took
// 3% of the time at 2^18), so a chunk makes few.
constexpr int kHeldTiles = 16;
inline int held_tiles(int longest)
{
    return longest < 2 * kHeldTiles ? kHeldTiles : longest > 128 ? 64 : longest / 2;
}

// Waves that share a one-wave block's chunk: the chunk partials of one-wave
// blocks were two thirds of what the fold reads (1 tile, 1 partial).  Forward
// calls with four waves to a partial against one: 86.7 -> 81.5 us at 18,000
// bodies, 144.9 -> 137.2 at 24,000, 218.7 -> 209.2 at 30,000.
constexpr int kTileSplit = 4;

// One-group plans of one-wave blocks of 64 K particles with at most one tile
// per wave (kTileSplit waves a workgroup), laid out in the workspace of a
// variant's own plan `pl`: false if it does not fit there.  C counts
// workgroups.  Sizes that take it, and what it replaces there: see
// forward_sym_run and run_backward_sym.
inline bool one_tile_plan(int64_t n, int K, const SymPlan &pl, SymPlan *out)
{
    SymPlan t = pl;
    t.M = (int)((n + 64 * K - 1) / (64 * K));
    t.G = t.M / 2;
    t.C = ((t.G + 1) * K + kTileSplit - 1) / kTileSplit;
    if (pl.groups != 1 || t.C + t.G > pl.C + pl.G) return false;
    *out = t;
    return true;
}
// Below kOneTileBegin the blocks of 256 particles these plans have are too few: see
// the same places.  They end where the plan of the forward's 4-wave four-row
// blocks ends: at M = 49 of its blocks it has 167 + 24 slots, and a tile per wave
// takes 195.
constexpr int kOneTileBegin = 10500, kOneTileEnd = 48 * 1024 + 1;

// Library workspace allowed for one pair-once evaluation of n particles
// (partials and running sum) before the ring is split into more groups:
// 1 GiB, or 16 float4 slots per particle where that is more (n > 2^22).
// The environment variable NBODY_SYM_WORKSPACE=<bytes> sets another limit
// (tests use it to split small rings into many groups).
inline size_t sym_workspace_budget(int64_t n)
{
    if (const char *env = std::getenv("NBODY_SYM_WORKSPACE")) {
        const unsigned long long v = std::strtoull(env, nullptr, 10);
        if (v > 0) return (size_t)v;
    }
    const size_t slots16 = 256 * (size_t)n;
    return slots16 > ((size_t)1 << 30) ? slots16 : ((size_t)1 << 30);
}

// Row groups that stand in for blocks of 128 particles (more ring offsets than
// slots that fit any small budget): refused exactly where sym_plan refuses, so that
// a workspace limit means the same at every size of a variant, ...
inline bool rows_refused(int64_t n, size_t budget) { return budget / (16 * (size_t)n) < 4; }

// ... though they take no workspace: asked for none, an arena still reports an
// injected allocation fault.
inline nbody_status rows_for_plan(const char *name, const Device &dev, int n, hipStream_t stream,
                                  const Arena &arena)
{
    const size_t budget = arena.budget(sym_workspace_budget(n));
    if (rows_refused(n, budget))
        return fail(NBODY_ERROR_INVALID_ARGUMENT,
                    "n = %d needs more than the %zu-byte workspace limit of %s", n, budget, name);
    void *none = nullptr;
    return arena.get(dev, stream, 0, &none);
}

// Number of tiles of block I in ring group [d_lo, d_hi): the TPB diagonal
// tiles when d_lo == 0, then TPB tiles per ring delta the block meets.
__host__ __device__ __forceinline__ int group_tiles(int I, int M, int d_lo, int d_hi, int TPB)
{
    const int dj = group_first_delta(d_lo);
    const int hi = min(d_hi - 1, ring_len(I, M));
    return (d_lo == 0 ? TPB : 0) + (hi >= dj ? (hi - dj + 1) * TPB : 0);
}

// Tile u of block I's sequence in ring group [d_lo, ...): the TPB diagonal
// tiles (delta 0) when the group holds them, then the ring tiles
// delta-major.  Returns the first particle index of the tile.
template <int PB>
__device__ __forceinline__ int tile_base(int u, int I, int M, int d_lo, int &delta)
{
    constexpr int TPB = PB / 64;
    if (d_lo == 0) {
        if (u < TPB) {
            delta = 0;
            return I * PB + u * 64;
        }
        u -= TPB;
    }
    const int q = u / TPB;
    delta = group_first_delta(d_lo) + q;
    int J = I + delta;
    if (J >= M) J -= M;
    return J * PB + (u - q * TPB) * 64;
}

__device__ __forceinline__ float4 load_particle(const float *__restrict__ x,
                                                const float *__restrict__ m, int j, int n)
{
    return (j < n) ? make_float4(x[3 * j], x[3 * j + 1], x[3 * j + 2], m[j])
                   : make_float4(kPadCol, kPadCol, kPadCol, 0.0f);
}

// One pair met once: i-side added to (tx, ty, tz, tp), j-side added to the
// slot value g (the chain of a step's K rows starts from the slot, so no
// separate add folds it in).  The slots hold +m_i r^3 d, the opposite of the
// j-side's force, which their readers negate: a negated factor here would
// take the long encoding.  POT false: the caller stores no potential, and its
// two terms (2 of the pair's 19 instructions) are not formed.
template <bool POT = true>
__device__ __forceinline__ void pair_once_fold(float xi, float yi, float zi, float mi, float4 q,
                                               float eps2, float &tx, float &ty, float &tz,
                                               float &tp, float4 &g)
{
    const float dx = xi - q.x;
    const float dy = yi - q.y;
    const float dz = zi - q.z;
    float s2 = __builtin_fmaf(dx, dx, eps2);
    s2 = __builtin_fmaf(dy, dy, s2);
    s2 = __builtin_fmaf(dz, dz, s2);
    const float r = __builtin_amdgcn_rsqf(s2);
    const float r3 = r * (r * r);
    const float f = q.w * r3;
    if (POT) tp = __builtin_fmaf(q.w, r, tp);
    tx = __builtin_fmaf(f, dx, tx);
    ty = __builtin_fmaf(f, dy, ty);
    tz = __builtin_fmaf(f, dz, tz);
    const float h = mi * r3;
    g.x = __builtin_fmaf(h, dx, g.x);
    g.y = __builtin_fmaf(h, dy, g.y);
    g.z = __builtin_fmaf(h, dz, g.z);
    if (POT) g.w = __builtin_fmaf(mi, r, g.w);
}

// pair_once_fold for the first R rows of a lane, the rows' reciprocal square roots
// taken as one group (rsq_group); the same operations in the same order.
// Whole calls, against K separate pair_once_fold: 215.5 -> 208.7 ms at 2^20
// bodies, 919 -> 907 us at 65,536, 69.1 -> 68.2 us at 16,384 without the
// potential.
template <int K, int R = K, bool POT = true, int B = 0>
__device__ __forceinline__ void pair_once_rows(const float (&xi)[K], const float (&yi)[K],
                                               const float (&zi)[K], const float (&mi)[K], float4 q,
                                               float eps2, float (&tx)[K], float (&ty)[K],
                                               float (&tz)[K], float (&tp)[K], float4 &g)
{
    constexpr int G = R < 4 ? R : 4;  // rows of this group (the first R rows in groups of four)
    float dx[G], dy[G], dz[G], r[G];
#pragma unroll
    for (int k = 0; k < G; ++k) {
        dx[k] = xi[B + k] - q.x;
        dy[k] = yi[B + k] - q.y;
        dz[k] = zi[B + k] - q.z;
        float s2 = __builtin_fmaf(dx[k], dx[k], eps2);
        s2 = __builtin_fmaf(dy[k], dy[k], s2);
        r[k] = __builtin_fmaf(dz[k], dz[k], s2);
    }
    rsq_group<G>(r);
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const float r3 = r[k] * (r[k] * r[k]);
        const float f = q.w * r3;
        if (POT) tp[B + k] = __builtin_fmaf(q.w, r[k], tp[B + k]);
        tx[B + k] = __builtin_fmaf(f, dx[k], tx[B + k]);
        ty[B + k] = __builtin_fmaf(f, dy[k], ty[B + k]);
        tz[B + k] = __builtin_fmaf(f, dz[k], tz[B + k]);
        const float h = mi[B + k] * r3;
        g.x = __builtin_fmaf(h, dx[k], g.x);
        g.y = __builtin_fmaf(h, dy[k], g.y);
        g.z = __builtin_fmaf(h, dz[k], g.z);
        if (POT) g.w = __builtin_fmaf(mi[B + k], r[k], g.w);
    }
    if constexpr (R > 4) {
        // the groups one after the other: their temporaries share registers
        __builtin_amdgcn_sched_barrier(0);
        pair_once_rows<K, R - 4, POT, B + 4>(xi, yi, zi, mi, q, eps2, tx, ty, tz, tp, g);
    }
}

// The 64 steps of a ring tile for one wave: lane l meets the particle in
// tile entry l + s at step s and adds its j-side terms to slot l + s.
// `tile` has kTileLds entries (the tile twice), `slot` this wave's
// kSlotLds slots.
// R < K: only the wave's first R row groups hold particles (the last block of
// a system); the others are padding with mass 0, whose terms are exactly zero
// on both sides, so skipping them changes no bit.
template <int K, int R = K, bool POT = true>
__device__ __forceinline__ void ring_tile_steps(const float (&xi)[K], const float (&yi)[K],
                                                const float (&zi)[K], const float (&mi)[K],
                                                const float4 *tile, float4 *slot, int lane,
                                                float eps2, float (&tx)[K], float (&ty)[K],
                                                float (&tz)[K], float (&tp)[K])
{
    const float4 *tq = tile + lane;
    float4 *sl = slot + lane;
    float4 q = tq[0];
    // about 600 to 1,200 operations per trip; few where the loop is one of K
    constexpr int kUnroll = R < K ? 2 : K > 8 ? 2 : K > 4 ? 4 : 8;
#pragma unroll kUnroll
    for (int s = 0; s < 64; ++s) {
        // Compiler-only barrier: this step's slot read stays after the
        // previous step's slot write (another lane wrote the slot read here).
        __asm__ volatile("" ::: "memory");
        float4 g = sl[s];
        const float4 qn = tq[s + 1];  // next step's particle (read-only tile)
        pair_once_rows<K, R, POT>(xi, yi, zi, mi, q, eps2, tx, ty, tz, tp, g);
        sl[s] = g;
        q = qn;
    }
    // particle e collected in slots e and e + 64: fold them into slot e
    __asm__ volatile("" ::: "memory");
    const float4 lo = slot[lane];
    const float4 hi = slot[lane + 64];
    slot[lane] = make_float4(lo.x + hi.x, lo.y + hi.y, lo.z + hi.z, lo.w + hi.w);
}

// ring_tile_steps with shorter slot chains, for blocks held with more rows per
// lane than the plan they come from (twice the rows, twice as long float32
// chains): the slots are emptied every kSlotSteps steps into the lane's sum of
// its tile particle.  Error of p against float64 (2-norm) at 65,536 bodies: four
// rows per lane 2.7e-8, eight 3.0e-8, eight so 2.6e-8; every 32 steps 2.7e-8.
// Whole calls take 1% longer.
constexpr int kSlotSteps = 16;

template <int K, bool POT>
__device__ __forceinline__ void ring_tile_short(const float (&xi)[K], const float (&yi)[K],
                                                const float (&zi)[K], const float (&mi)[K],
                                                const float4 *tile, float4 *slot, int lane,
                                                float eps2, float (&tx)[K], float (&ty)[K],
                                                float (&tz)[K], float (&tp)[K])
{
    const float4 *tq = tile + lane;
    float4 *sl = slot + lane;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 q = tq[0], sum = zero;
#pragma nounroll
    for (int h = 0; h < 64 / kSlotSteps; ++h) {
        constexpr int kUnroll = K > 4 ? 4 : 8;
#pragma unroll kUnroll
        for (int s = 0; s < kSlotSteps; ++s) {
            // as in ring_tile_steps
            __asm__ volatile("" ::: "memory");
            float4 g = sl[s];
            const float4 qn = tq[s + 1];
            pair_once_rows<K, K, POT>(xi, yi, zi, mi, q, eps2, tx, ty, tz, tp, g);
            sl[s] = g;
            q = qn;
        }
        tq += kSlotSteps;
        sl += kSlotSteps;
        __asm__ volatile("" ::: "memory");
        const float4 lo = slot[lane];
        const float4 hi = slot[lane + 64];
        sum.x += lo.x + hi.x;
        sum.y += lo.y + hi.y;
        sum.z += lo.z + hi.z;
        sum.w += lo.w + hi.w;
        slot[lane] = zero;
        slot[lane + 64] = zero;
    }
    __asm__ volatile("" ::: "memory");
    slot[lane] = sum;
}

// ring_tile_steps of the first kv < K row groups.
template <int K, int R, bool POT>
__device__ __forceinline__ void ring_tile_some(int kv, const float (&xi)[K], const float (&yi)[K],
                                               const float (&zi)[K], const float (&mi)[K],
                                               const float4 *tile, float4 *slot, int lane,
                                               float eps2, float (&tx)[K], float (&ty)[K],
                                               float (&tz)[K], float (&tp)[K])
{
    if constexpr (R > 0) {
        if (kv == R)
            ring_tile_steps<K, R, POT>(xi, yi, zi, mi, tile, slot, lane, eps2, tx, ty, tz, tp);
        else
            ring_tile_some<K, R - 1, POT>(kv, xi, yi, zi, mi, tile, slot, lane, eps2, tx, ty, tz, tp);
    }
}

// One step s of a diagonal tile: rows k < R meet entry l + s pair-once.
template <int K, int R, bool POT = true>
__device__ __forceinline__ void diag_step(const float (&xi)[K], const float (&yi)[K],
                                          const float (&zi)[K], const float (&mi)[K],
                                          const float4 *tq, float4 *sl, int s, float eps2,
                                          float (&tx)[K], float (&ty)[K], float (&tz)[K],
                                          float (&tp)[K])
{
    if constexpr (R > 0) {
        static_assert(R <= 4, "one group of rows");
        // keep this step's slot read after the previous step's slot write
        __asm__ volatile("" ::: "memory");
        const float4 q = tq[s];
        float4 g = sl[s];
        pair_once_rows<K, R, POT>(xi, yi, zi, mi, q, eps2, tx, ty, tz, tp, g);
        sl[s] = g;
    }
}

// Diagonal tile whose rows are this wave's row group KT (rows k < KT belong
// to earlier tiles of the block and meet it pair-once; rows k > KT to later
// ones, which meet it from their side).  Row group KT meets its own tile
// pair-once too: lane l and particle l + s (mod 64) form each unordered
// pair once for s = 1..31, and for s = 32 the pair {l, l + 32} is met by
// both lanes, so each takes its i-side only; s = 0 (the particle itself)
// and s = 33..63 (met as 64 - s by the partner) are skipped.  The j-side
// sums fill this wave's slots like a ring tile's and are folded to slot e.
template <int K, int KT, bool POT = true>
__device__ __forceinline__ void diag_self_steps(const float (&xi)[K], const float (&yi)[K],
                                                const float (&zi)[K], const float (&mi)[K],
                                                const float4 *tile, float4 *slot, int lane,
                                                float eps2, float (&tx)[K], float (&ty)[K],
                                                float (&tz)[K], float (&tp)[K])
{
    const float4 *tq = tile + lane;
    float4 *sl = slot + lane;
    // The loops run two steps per trip and are kept rolled: fully unrolled,
    // the K instances of this function made a kernel larger than the
    // instruction cache and slowed its ring loop.
    diag_step<K, KT, POT>(xi, yi, zi, mi, tq, sl, 0, eps2, tx, ty, tz, tp);
#pragma nounroll
    for (int s = 1; s < 31; s += 2) {
        diag_step<K, KT + 1, POT>(xi, yi, zi, mi, tq, sl, s, eps2, tx, ty, tz, tp);
        diag_step<K, KT + 1, POT>(xi, yi, zi, mi, tq, sl, s + 1, eps2, tx, ty, tz, tp);
    }
    diag_step<K, KT + 1, POT>(xi, yi, zi, mi, tq, sl, 31, eps2, tx, ty, tz, tp);
    diag_step<K, KT, POT>(xi, yi, zi, mi, tq, sl, 32, eps2, tx, ty, tz, tp);
    pair_term(xi[KT], yi[KT], zi[KT], tq[32], eps2, tx[KT], ty[KT], tz[KT], tp[KT]);
    if (KT > 0) {
#pragma nounroll
        for (int s = 33; s < 63; s += 2) {
            diag_step<K, KT, POT>(xi, yi, zi, mi, tq, sl, s, eps2, tx, ty, tz, tp);
            diag_step<K, KT, POT>(xi, yi, zi, mi, tq, sl, s + 1, eps2, tx, ty, tz, tp);
        }
        diag_step<K, KT, POT>(xi, yi, zi, mi, tq, sl, 63, eps2, tx, ty, tz, tp);
    }
    __asm__ volatile("" ::: "memory");
    const float4 lo = slot[lane];
    const float4 hi = slot[lane + 64];
    slot[lane] = make_float4(lo.x + hi.x, lo.y + hi.y, lo.z + hi.z, lo.w + hi.w);
}

template <int K, int KT = 0, bool POT = true>
__device__ __forceinline__ void diag_tile_dispatch(int kt, const float (&xi)[K],
                                                   const float (&yi)[K], const float (&zi)[K],
                                                   const float (&mi)[K], const float4 *tile,
                                                   float4 *slot, int lane, float eps2,
                                                   float (&tx)[K], float (&ty)[K], float (&tz)[K],
                                                   float (&tp)[K])
{
    if (kt == KT)
        diag_self_steps<K, KT, POT>(xi, yi, zi, mi, tile, slot, lane, eps2, tx, ty, tz, tp);
    else if constexpr (KT + 1 < K)
        diag_tile_dispatch<K, KT + 1, POT>(kt, xi, yi, zi, mi, tile, slot, lane, eps2, tx, ty, tz, tp);
}

// The 64 steps of diagonal tile t for one wave of a wider block.  Lane l meets
// tile particle (l + s) mod 64 at step s: row tile a = a0 + k meets it
// pair-once if a < t, as masked ordered pairs if a == t, not at all if a > t.
// j-side sums go to this wave's LDS slots (read-modify-write).
template <int K>
__device__ __forceinline__ void diag_tile_steps(const float (&xi)[K], const float (&yi)[K],
                                                const float (&zi)[K], const float (&mi)[K],
                                                const int (&ii)[K], const float4 *tile,
                                                float4 *slot, int lane, int a0, int t, int jbase,
                                                float eps2, float (&tx)[K], float (&ty)[K],
                                                float (&tz)[K], float (&tp)[K])
{
    const bool any_once = a0 < t;
    float4 q = tile[lane];
    for (int s = 0; s < 64; ++s) {
        const int jj = (lane + s) & 63;
        // Compiler-only barrier: this step's slot read stays after the
        // previous step's slot write (another lane may have written it).
        __asm__ volatile("" ::: "memory");
        float4 g = make_float4(0.f, 0.f, 0.f, 0.f);
        if (any_once) g = slot[jj];
        const float4 qn = tile[(jj + 1) & 63];  // next step's particle (read-only tile)
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (a0 + k < t)
                pair_once_fold<true>(xi[k], yi[k], zi[k], mi[k], q, eps2, tx[k], ty[k], tz[k],
                                     tp[k], g);
            else if (a0 + k == t)
                pair_term_masked(xi[k], yi[k], zi[k], q, eps2, jbase + jj == ii[k], tx[k], ty[k],
                                 tz[k], tp[k]);
        }
        if (any_once) slot[jj] = g;
        q = qn;
    }
}

// LDS entries of one wave of a tile-split workgroup: the tile and the slots,
// and at the end K <= 4 rows of row sums.
constexpr int kWaveLds = kTileLds + kSlotLds;

// LDS buffers of a pair-once workgroup: blocks of several waves keep two tiles
// and two sets of slots, so that one barrier per tile suffices; a one-wave
// block needs no barrier, and its single set leaves room for more workgroups.
template <int W>
constexpr int kSymBuffers = W > 1 ? 2 : 1;

// One workgroup of W*64 lanes evaluates chunk c of block I.  x, m and
// partial are the system's own arrays (offsets already applied).  tile
// (kSymBuffers<W> tiles) and jacc (kSymBuffers<W> sets of W slot arrays) are
// the workgroup's LDS buffers.  Blocks of several waves start with a workgroup
// barrier, so their LDS buffers may be reused by consecutive calls; one-wave
// blocks (T == 1) need none.  With T > 1 there is no barrier after the last reads
// of other waves' regions: a caller puts one between two calls (the ticket loop
// of batched_sym_dyn_kernel has it).
//
// Diagonal tiles are pair-once too (for W <= 8; larger blocks meet them as
// masked ordered pairs): the rows of lane-slot k of wave wv form
// the block's tile a = wv*K + k.  On diagonal tile t, row tile a < t meets
// it pair-once, a == t meets it as ordered pairs with j == i removed by
// index (one-wave blocks: pair-once within the tile, diag_self_steps), and
// a > t skips it (that pair of tiles is met on diagonal tile a).
// The j-side sums of a diagonal tile belong to rows of the same block; the
// wave that holds tile t's rows adds them to its own accumulators.
// POT false: no potential is stored, and the ring and one-wave diagonal
// tiles do not form its terms (the partials' w component is then partial).
// SKIP_PAD (ensembles): skip the ring-tile work of row groups that hold only padding
// (bitwise neutral: their terms are exactly zero).  Worth it for ensembles
// of small systems, where a last block is often part padding (5% of the
// row-group work on the 4,096-system ensemble); single systems keep the
// lighter loop.
//
// Blocks of several waves pass one barrier per tile: while a wave takes the
// steps of tile b, the next tile is staged in the other buffer; after the
// barrier every wave clears its slots of the other set (whose sums were read
// before the barrier) and all threads share the sum of the W slot sets, one
// component each.
//
// HELD: chunks of more than held_tiles tiles hand their sums over in between.
// SHORT: ring_tile_short.
//
// T > 1 (one-wave blocks): T waves of a workgroup hold the same rows and take
// one of T consecutive sub-chunks of chunk c each, with an LDS region of
// kWaveLds entries per wave (its tile, then its slots) from `tile` on; their
// row sums are added in wave order (in float64) at the end, so that a chunk writes
// (and the fold reads) one partial for T waves' tiles.  (Ensembles, one chunk per block:
// every T-th tile each.)
template <int W, int K, bool SKIP_PAD = false, bool POT = true, int T = 1, bool SHORT = false,
          bool HELD = T == 1 && !SKIP_PAD>
__device__ __forceinline__ void pair_once_block(const float *__restrict__ x,
                                                const float *__restrict__ m, int n, float eps2,
                                                int M, int I, int c, int C, int d_lo, int d_hi,
                                                float4 *partial, float4 *tile,
                                                float4 (*jacc)[kSlotLds], int held_tiles = 0)
{
    constexpr int PB = W * 64 * K;   // particles per block
    constexpr int TPB = PB / 64;     // 64-particle tiles per block
    constexpr int NB = kSymBuffers<W>;
    static_assert(T == 1 || (W == 1 && K * 64 <= kWaveLds), "a tile split is of one-wave blocks");
    const int lane = threadIdx.x & 63;
    const int tw = T > 1 ? (int)(threadIdx.x >> 6) : 0;  // which of T sub-chunks
    const int tid = T > 1 ? lane : (int)threadIdx.x;     // thread of the block's W waves
    const int wv = tid >> 6;
    float4 *const lds = tile;
    if (T > 1) {
        tile = lds + tw * kWaveLds;
        jacc = reinterpret_cast<float4(*)[kSlotLds]>(tile + kTileLds);
    }
    // One wave's LDS accesses complete in issue order: between its lanes a
    // compiler barrier is enough.
    const auto block_sync = [&]() {
        if (W == 1)
            __asm__ volatile("" ::: "memory");
        else
            __syncthreads();
    };

    // ---- own rows
    float xi[K], yi[K], zi[K], mi[K];
    int ii[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = I * PB + wv * 64 * K + k * 64 + lane;
        ii[k] = i;
        if (i < n) {
            xi[k] = x[3 * i];
            yi[k] = x[3 * i + 1];
            zi[k] = x[3 * i + 2];
            mi[k] = m[i];
        } else {
            xi[k] = yi[k] = zi[k] = kPadRow;
            mi[k] = 0.0f;
        }
    }
    float ax[K], ay[K], az[K], ap[K];
#pragma unroll
    for (int k = 0; k < K; ++k) ax[k] = ay[k] = az[k] = ap[k] = 0.0f;
    // row groups of this wave that hold particles (K except in a last block)
    const int kv = SKIP_PAD ? min(K, max(0, (n - (I * PB + wv * 64 * K) + 63) / 64)) : K;

    // ---- this chunk's share of the block's tile sequence in the group;
    // tiles that hold only padding are skipped (uniform).
    const int U = group_tiles(I, M, d_lo, d_hi, TPB);
    const int dj = group_first_delta(d_lo);
    // (a small system's one chunk: every T-th tile, cheap diagonal ones evenly)
    constexpr bool kStride = T > 1 && SKIP_PAD;
    constexpr int kStep = kStride ? T : 1;
    const int u0 = kStride ? tw : chunk_begin(U, C * T, c * T + tw);
    const int u1 = kStride ? U : chunk_begin(U, C * T, c * T + tw + 1);
    // Small workgroups prefetch the next tile into registers while the
    // current one is consumed; 16-wave blocks (one per CU, 128 VGPRs) have
    // no registers to spare and rely on the other waves to hide the load.
    constexpr bool kPrefetch = (W <= 8);
    // Diagonal tiles pair-once (halves their work) where registers allow;
    // 16-wave blocks meet them as masked ordered pairs (at 2^17 particles
    // and up the diagonal is under 1/32 of the pairs).
    constexpr bool kOnceDiag = (W <= 8);
    // One-wave blocks (ensembles of small systems, mid-size single systems,
    // where diagonal tiles are a fifth of the work) also meet each diagonal
    // tile's own 64 particles pair-once (diag_self_steps).  Wider blocks
    // keep the masked ordered self tile: there the diagonal is rare, and
    // the larger code changed the schedule of their ring loop (6-8% slower
    // at 2^20 bodies).
    constexpr bool kSelfDiag = (W == 1 && K <= 4);
    int u = u0, delta = 0, jbase = 0;
    for (; u < u1; u += kStep)
        if ((jbase = tile_base<PB>(u, I, M, d_lo, delta)) < n) break;
    float4 next = make_float4(0.f, 0.f, 0.f, 0.f);
    if (kPrefetch && u < u1 && tid < 64) next = load_particle(x, m, jbase + tid, n);
    in_vgpr(eps2);
    // The rows have arrived here, so that no wait for them in the tile loop
    // also waits for the prefetch.
#pragma unroll
    for (int k = 0; k < K; ++k)
        __asm__ volatile("" : "+v"(xi[k]), "+v"(yi[k]), "+v"(zi[k]), "+v"(mi[k]));

    const auto stage = [&](int b) {
        if (tid < 64) {
            const float4 v = kPrefetch ? next : load_particle(x, m, jbase + tid, n);
            tile[b * kTileLds + tid] = v;
            tile[b * kTileLds + tid + 64] = v;
        }
    };
    const auto clear_slots = [&](int b) {
        jacc[b * W + wv][lane] = make_float4(0.f, 0.f, 0.f, 0.f);
        jacc[b * W + wv][lane + 64] = make_float4(0.f, 0.f, 0.f, 0.f);
    };
    // the tile after the current one, and its load
    const auto advance = [&]() {
        for (u += kStep; u < u1; u += kStep)
            if ((jbase = tile_base<PB>(u, I, M, d_lo, delta)) < n) break;
        if (kPrefetch && u < u1 && tid < 64) next = load_particle(x, m, jbase + tid, n);
    };

    // The row sums so far, added to the chunk's partial: at the end, and every
    // held_tiles tiles before (HELD).
    [[maybe_unused]] int held = 0;
    bool fresh = true;
    const auto hand_over = [&]() {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (ii[k] < n) {
                float4 *out = partial + (size_t)c * n + ii[k];
                float4 v = make_float4(ax[k], ay[k], az[k], ap[k]);
                if (!fresh) {
                    const float4 w = *out;
                    v = make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
                }
                *out = v;
            }
            ax[k] = ay[k] = az[k] = ap[k] = 0.0f;
        }
        held = 0;
        fresh = false;
    };

    int b = 0;
    if (NB == 2 && u < u1) {
        __syncthreads();  // the LDS buffers are free
        stage(0);
        clear_slots(0);
        __syncthreads();
    }
    while (u < u1) {
        if (NB == 1) {
            // the previous tile and its slot sums are done
            block_sync();
            stage(0);
            clear_slots(0);
            block_sync();
        }
        const int cur_u = u, cur_delta = delta, cur_base = jbase;
        advance();

        float tx[K], ty[K], tz[K], tp[K];
#pragma unroll
        for (int k = 0; k < K; ++k) tx[k] = ty[k] = tz[k] = tp[k] = 0.0f;

        const int t = cur_u;                         // diagonal tile index when cur_delta == 0
        const bool diag = (cur_delta == 0);
        const float4 *cur_tile = tile + b * kTileLds;
        float4 *slot = &jacc[b * W + wv][0];
        if (!diag) {
            if constexpr (SHORT)
                ring_tile_short<K, POT>(xi, yi, zi, mi, cur_tile, slot, lane, eps2, tx, ty, tz, tp);
            else if (!SKIP_PAD || kv == K)
                ring_tile_steps<K, K, POT>(xi, yi, zi, mi, cur_tile, slot, lane, eps2, tx, ty, tz, tp);
            else
                ring_tile_some<K, K - 1, POT>(kv, xi, yi, zi, mi, cur_tile, slot, lane, eps2, tx, ty,
                                              tz, tp);
        } else if constexpr (kSelfDiag) {
            // one wave: its row group k is the block's tile k, so diagonal
            // tile t meets row groups k < t pair-once and row group t itself
            diag_tile_dispatch<K, 0, POT>(t, xi, yi, zi, mi, cur_tile, slot, lane, eps2, tx, ty, tz,
                                          tp);
        } else if (kOnceDiag) {
            diag_tile_steps<K>(xi, yi, zi, mi, ii, cur_tile, slot, lane, wv * K, t, cur_base, eps2, tx,
                               ty, tz, tp);
        } else {
            // ordered pairs, i-side only, j == i removed by index
            for (int s = 0; s < 64; ++s) {
                const float4 q = cur_tile[s];
                const int j = cur_base + s;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    pair_term_masked(xi[k], yi[k], zi[k], q, eps2, j == ii[k], tx[k], ty[k], tz[k],
                                     tp[k]);
            }
        }
        __asm__ volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < K; ++k) {
            ax[k] += tx[k];
            ay[k] += ty[k];
            az[k] += tz[k];
            ap[k] += tp[k];
        }
        if (NB == 2 && u < u1) stage(b ^ 1);
        block_sync();  // every wave's j-side slots are complete
        if (NB == 2 && u < u1) clear_slots(b ^ 1);
        // every wave left particle e's sums in its slot e (components xyz with
        // the opposite sign); they are added in wave order
        if (!diag) {
            float4 *out = partial + (size_t)(C + cur_delta - dj) * n + cur_base;
            if constexpr (W == 1) {
                const float4 sum = jacc[0][tid];
                if (cur_base + tid < n) out[tid] = make_float4(-sum.x, -sum.y, -sum.z, sum.w);
            } else {
                for (int f = tid; f < 256; f += W * 64) {
                    float sum = reinterpret_cast<const float *>(jacc[b * W])[f];
#pragma unroll
                    for (int w2 = 1; w2 < W; ++w2)
                        sum += reinterpret_cast<const float *>(jacc[b * W + w2])[f];
                    if (cur_base + (f >> 2) < n)
                        reinterpret_cast<float *>(out)[f] = (f & 3) == 3 ? sum : -sum;
                }
            }
        } else if (kOnceDiag && wv == t / K) {
            // this wave holds diagonal tile t's rows (lane-slot t % K)
            float4 sum = jacc[b * W][lane];
#pragma unroll
            for (int w2 = 1; w2 < W; ++w2) {
                const float4 v = jacc[b * W + w2][lane];
                sum.x += v.x;
                sum.y += v.y;
                sum.z += v.z;
                sum.w += v.w;
            }
            const int kt = t - wv * K;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (k == kt) {
                    ax[k] -= sum.x;
                    ay[k] -= sum.y;
                    az[k] -= sum.z;
                    ap[k] += sum.w;
                }
        }
        if (NB == 2) b ^= 1;
        if (HELD && ++held == held_tiles) hand_over();
    }

    if constexpr (T == 1) {
        hand_over();
    } else {
        // the T waves' row sums through their own LDS regions, one component
        // of every 64 T / 4 rows per thread
        __asm__ volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < K; ++k) tile[k * 64 + lane] = make_float4(ax[k], ay[k], az[k], ap[k]);
        __syncthreads();
        float *out = reinterpret_cast<float *>(partial + (size_t)c * n + I * PB);
        const float *all = reinterpret_cast<const float *>(lds);
        for (int f = threadIdx.x; f < K * 256; f += T * 64) {
            double sum = all[f];
#pragma unroll
            for (int w = 1; w < T; ++w) sum += all[w * kWaveLds * 4 + f];
            if (I * PB + (f >> 2) < n) out[f] = (float)sum;
        }
    }
}

}  // namespace nbody
