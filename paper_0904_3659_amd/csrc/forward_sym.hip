// Forward evaluation of Eq. (gravity) (Sec. I) with every unordered pair
// computed once (see pair_once.hpp for the block/ring decomposition, the
// LDS slot sums and the partial layout).  Grid: one workgroup per (block I,
// chunk c); a second kernel adds each particle's partial slots.
#include "pair_once.hpp"

namespace nbody {
namespace {

struct SymArgs {
    const float *x;
    const float *m;
    int n;
    float eps2;
    int M;            // blocks
    int C;            // chunks per block
    int d_lo, d_hi;   // ring deltas of this launch's group
    float4 *partial;  // [C + G][n]
    int held;         // held_tiles of the longest chunk
};

// Waves per workgroup: those of a block, or those that split a one-wave
// block's tiles.
template <int W>
constexpr int kSymSplit = W == 1 ? kTileSplit : 1;
template <int W>
constexpr int kSymThreads = 64 * W * kSymSplit<W>;

template <int W, int K, bool POT, bool SHORT = false, bool HELD = W != 1>
__global__ __launch_bounds__(kSymThreads<W>, K == 8 ? 3 : 1) void forward_sym_kernel(SymArgs A)
{
    const int c = blockIdx.x / A.M;  // chunk-major (chunk_begin)
    const int I = blockIdx.x - c * A.M;
    if constexpr (W == 1) {
        __shared__ float4 lds[kTileSplit * kWaveLds];
        pair_once_block<1, K, false, POT, kTileSplit, SHORT>(A.x, A.m, A.n, A.eps2, A.M, I, c, A.C, A.d_lo,
                                                      A.d_hi, A.partial, lds, nullptr);
    } else {
        __shared__ float4 tile[kSymBuffers<W> * kTileLds];
        __shared__ float4 jacc[kSymBuffers<W> * W][kSlotLds];
        pair_once_block<W, K, false, POT, 1, SHORT, HELD>(A.x, A.m, A.n, A.eps2, A.M, I, c, A.C, A.d_lo, A.d_hi,
                                          A.partial, tile, jacc, A.held);
    }
}

// Workgroups of W waves per CU (counting each wave of a tile split as one).
template <int W, int K>
nbody_status sym_occupancy(int *per_cu)
{
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        per_cu, forward_sym_kernel<W, K, true>, kSymThreads<W>, 0);
    if (e != hipSuccess) return hip_fail(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    if (*per_cu < 1) *per_cu = 1;
    *per_cu *= kSymSplit<W>;
    return NBODY_OK;
}

// The launches of a plan whose blocks are W waves x K rows per lane.
template <int W, int K, bool SHORT, bool HELD = W != 1>
nbody_status launch_sym(const SymPlan &pl, void *ws, const char *name, const float *x,
                        const float *m, int n, float eps2, float *a, float *p, hipStream_t stream,
                        const LfEpi *epi, bool *fused)
{
    constexpr int PB = W * 64 * K;
    float4 *partial = static_cast<float4 *>(ws);
    double4 *acc = pl.acc_bytes ? reinterpret_cast<double4 *>(static_cast<char *>(ws) + pl.partial_bytes)
                                : nullptr;
    if (fault_injected("launch")) return fail(NBODY_ERROR_LAUNCH_FAILED, "injected launch fault");
    const bool lf = epi && epi->mode != kLfNone;
    const int C = pl.C, held = held_tiles(longest_chunk(pl, W * K));
    for (int g = 0; g < pl.groups; ++g) {
        SymArgs A{x, m, n, eps2, pl.M, C, 0, 0, partial, held};
        sym_group(pl, g, &A.d_lo, &A.d_hi);
        prof_mark(stream, 0);
        if (p)
            hipLaunchKernelGGL((forward_sym_kernel<W, K, true, SHORT, HELD>), dim3(pl.M * C),
                               dim3(kSymThreads<W>), 0, stream, A);
        else
            hipLaunchKernelGGL((forward_sym_kernel<W, K, false, SHORT, HELD>), dim3(pl.M * C),
                               dim3(kSymThreads<W>), 0, stream, A);
        prof_mark(stream, 1);
        nbody_status st = check_launch(name);
        if (st != NBODY_OK) return st;
        const int first = g == 0, last = g == pl.groups - 1;
        if (last && lf)
            hipLaunchKernelGGL((slot_fold_kernel<PB, true>), dim3((n + 63) / 64), dim3(256), 0,
                               stream, partial, n, pl.M, C, A.d_lo, A.d_hi, first, last, acc, a,
                               p, *epi);
        else
            hipLaunchKernelGGL((slot_fold_kernel<PB>), dim3((n + 63) / 64), dim3(256), 0, stream,
                               partial, n, pl.M, C, A.d_lo, A.d_hi, first, last, acc, a, p,
                               LfEpi{});
        st = check_launch("slot_fold");
        if (st != NBODY_OK) return st;
    }
    if (lf && fused) *fused = true;
    return NBODY_OK;
}

// OCC divides the chunk count: 1 fills every resident workgroup slot once;
// 2 gives half as many, twice as long workgroups (fewer partial slots, less
// tail imbalance at small n, lower occupancy).  ROUNDS multiplies it: that
// many rounds of shorter workgroups (down to one tile each), which the
// hardware dispatcher hands out as slots free up, evening out the tail of
// a grid whose workgroups hold only a few tiles.
// The kernel may hold a block of W waves x K rows as KW waves x KK rows (the
// same P = 64 W K particles and the same plan).
template <int W, int K, int OCC, int ROUNDS = 1, int KW = W, int KK = K>
nbody_status run_sym(const char *name, const Device &dev, const float *x, const float *m, int n,
                     float eps2, float *a, float *p, hipStream_t stream, const LfEpi *epi,
                     bool *fused, const Arena &arena)
{
    static_assert(KW * KK == W * K, "the same block");
    constexpr int PB = W * 64 * K;
    if constexpr (W == 1 && K == 2) {
        if (row_band(n)) {
            // refused where the plan of many ring offsets would be; no workspace
            const nbody_status st = rows_for_plan(name, dev, n, stream, arena);
            return st != NBODY_OK ? st
                                  : forward_rows_run(1, name, dev, x, m, n, eps2, a, p, stream, epi, fused);
        }
    }
    int per_cu = 0;
    // sized by the kernel that forms the potential, also when p is not
    // stored: the same plan keeps a bitwise the same either way
    nbody_status st = sym_occupancy<W, K>(&per_cu);
    if (st != NBODY_OK) return st;
    SymPlan pl;
    if (!sym_plan(n, PB, (int64_t)per_cu * dev.num_cu * ROUNDS, OCC,
                  arena.budget(sym_workspace_budget(n)), &pl))
        return fail(NBODY_ERROR_INVALID_ARGUMENT,
                    "n = %d needs more than the %zu-byte workspace limit of %s", n,
                    arena.budget(sym_workspace_budget(n)), name);
    void *ws = nullptr;
    st = arena.get(dev, stream, pl.bytes(), &ws);
    if (st != NBODY_OK) return st;
    // A tile per one-wave block of 256 particles.  Calls with the potential, row
    // groups / a tile per wave: 32.2 / 34.7 us at 10,000 bodies, 35.2 / 35.4 at
    // 10,499, 38.7 / 35.7 at 11,000, 44.5 / 42.8 at 12,000; planned chunks of 2-4
    // tiles / a tile per wave (both with longer slot chains): 50.7 / 47.9 at 13,000,
    // 71.5 / 69.2 at 16,384, the same from 18,000 to 30,000 (there the plan has a
    // tile per wave), 246 / 233 at 33,000, 341 / 325 at 39,000; four waves' blocks of
    // 1,024 / a tile per wave: 373 / 354 at 40,000, 443 / 439 at 45,000, 500 / 497 at
    // 48,000.
    if constexpr (W == 1 || (W == 4 && K == 4 && KW == 4)) {
        SymPlan one;
        if (n >= kOneTileBegin && n < kOneTileEnd && one_tile_plan(n, 4, pl, &one))
            return launch_sym<1, 4, (4 > K)>(one, ws, name, x, m, n, eps2, a, p, stream, epi, fused);
    }
    if (KW == 1) pl.C = (pl.C + kTileSplit - 1) / kTileSplit;  // counted in workgroups
    // Two-wave blocks of 1,024 keep at most 72 chunks (partials to write and fold
    // per row; the rows' running sums then span up to 16 tiles).  As planned / 96 / 72 / 52: 541 / 524 / 521 / 558 us at 50,000
    // bodies (168 planned), 709 / 699 / 688 / 717 at 60,000, 823 / 819 / 807 /
    // 820 at 65,536, 1203 / 1205 / 1195 / 1196 at 80,000.
    if constexpr (KW == 2 && KK == 8 && ROUNDS > 1) {
        if (pl.C > 72) pl.C = 72;
        // short chunks (up to some 110,000 bodies) hand nothing over in between:
        // 1% less time at 65,536 bodies without that code
        if (longest_chunk(pl, KW * KK) <= kHeldTiles)
            return launch_sym<KW, KK, (KK > K), false>(pl, ws, name, x, m, n, eps2, a, p, stream, epi,
                                                       fused);
    }
    // (4-wave eight-row blocks, of 2^20 bodies and more: their chunks are so long that
    // handing over alone takes more off the error than longer slot chains add)
    return launch_sym<KW, KK, (KK > K && KW < 4)>(pl, ws, name, x, m, n, eps2, a, p, stream, epi, fused);
}

}  // namespace

nbody_status forward_sym_occupancy(int W, int K, int *per_cu)
{
    if (W == 8 && K == 4) return sym_occupancy<8, 4>(per_cu);
    if (W == 4 && K == 8) return sym_occupancy<4, 8>(per_cu);
    if (W == 4 && K == 4) return sym_occupancy<4, 4>(per_cu);
    if (W == 2 && K == 8) return sym_occupancy<2, 8>(per_cu);
    if (W == 16 && K == 4) return sym_occupancy<16, 4>(per_cu);
    if (W == 2 && K == 4) return sym_occupancy<2, 4>(per_cu);
    if (W == 1 && K == 4) return sym_occupancy<1, 4>(per_cu);
    if (W == 1 && K == 2) return sym_occupancy<1, 2>(per_cu);
    if (W == 2 && K == 2) return sym_occupancy<2, 2>(per_cu);
    if (W == 4 && K == 2) return sym_occupancy<4, 2>(per_cu);
    return fail(NBODY_ERROR_INTERNAL, "no pair-once forward kernel for W=%d K=%d", W, K);
}

nbody_status forward_sym_run(int W, int K, int occ, int rounds, const char *name,
                             const Device &dev, const float *x, const float *m, int n, float eps2,
                             float *a, float *p, hipStream_t stream, const LfEpi *epi, bool *fused,
                             const Arena &arena)
{
    if (rounds == 8) {
        if (W == 1 && K == 4 && occ == 1) return run_sym<1, 4, 1, 8>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
        if (W == 1 && K == 2 && occ == 1) return run_sym<1, 2, 1, 8>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
        // Eight rows per lane halve the LDS reads and writes per pair against
        // four (the two take turns in groups of four, so three waves per SIMD
        // still fit).  Sustained calls (before the sums of eight rows were cut
        // shorter, which takes 0.5-1.5%; above 110,000 bodies 2-3%): 8 x 4 as 4 x 8
        // 220.1 -> 212.5 ms at 2^20 bodies; 4 x 4 as 2 x 8 874 -> 860 us at 65,536,
        // 1975 -> 1947 at 100,000, but 358 -> 363 at 40,000, where the workgroups
        // are too few.  4 x 4 in equal chunks, one barrier more per tile, against 2 x 8
        // with the shorter sums: 14.2 / 12.6 ms at 2^18, 145 / 136 at 850,000.  Below
        // kOneTileEnd a tile per wave is level or ahead (run_sym).
        if (W == 4 && K == 4 && occ == 1 && n >= kOneTileEnd) return run_sym<4, 4, 1, 8, 2, 8>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
        if (W == 4 && K == 4 && occ == 1) return run_sym<4, 4, 1, 8>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
        if (W == 8 && K == 4 && occ == 1) return run_sym<8, 4, 1, 8, 4, 8>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
        return fail(NBODY_ERROR_INTERNAL, "no pair-once forward kernel for W=%d K=%d occ=%d rounds=%d", W, K, occ, rounds);
    }
    if (W == 8 && K == 4 && occ == 1) return run_sym<8, 4, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 8 && K == 4 && occ == 2) return run_sym<8, 4, 2>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 4 && K == 8 && occ == 1) return run_sym<4, 8, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 4 && K == 4 && occ == 1) return run_sym<4, 4, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 2 && K == 8 && occ == 1) return run_sym<2, 8, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 16 && K == 4 && occ == 1) return run_sym<16, 4, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 2 && K == 4 && occ == 1) return run_sym<2, 4, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 1 && K == 4 && occ == 1) return run_sym<1, 4, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 1 && K == 2 && occ == 1) return run_sym<1, 2, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 2 && K == 2 && occ == 1) return run_sym<2, 2, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    if (W == 4 && K == 2 && occ == 1) return run_sym<4, 2, 1>(name, dev, x, m, n, eps2, a, p, stream, epi, fused, arena);
    return fail(NBODY_ERROR_INTERNAL, "no pair-once forward kernel for W=%d K=%d occ=%d", W, K, occ);
}

}  // namespace nbody
