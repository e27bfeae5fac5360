// Backward (vector-Jacobian product) of Eq. (gravity) (Sec. I), float32 on
// gfx950.  For upstream weights w = dL/da and v = dL/dp the gradient of
// L = sum_i w_i . a_i + v_i p_i, gathered per output row k over j != k with
// d = x_k - x_j, r = (|d|^2 + eps2)^(-1/2), is
//     dL/dx_k = sum_j r^3 c_kj - r^3 (3 r^2 (c_kj . d) + b_kj) d,
//     dL/dm_k = sum_j r v_j - r^3 (w_j . d),
// with c_kj = m_j w_k - m_k w_j and b_kj = m_j v_k + m_k v_j.  The first
// sum is split as
//     sum_j r^3 c_kj = w_k A_k - m_k B_k,  A_k = sum_j m_j r^3,
//                                          B_k = sum_j r^3 w_j,
// so that the per-pair work is about 30 VALU operations and one v_rsq_f32.
//
// Decomposition as in the forward kernel: K rows per lane in VGPRs, j-tiles
// of BLOCK particles staged in LDS as two float4 per particle, (x, y, z, m)
// and (w_x, w_y, w_z, v); j-splits with a fixed-order reduction when the
// row count alone cannot fill the device; per-tile partial sums folded into
// the running sums (two-level accumulation).  No atomics.
#include "common.hpp"
#include "pair_once.hpp"
#include "wave_sum.hpp"

#include <cstring>
#include <type_traits>

namespace nbody {
namespace {

struct BwdArgs {
    const float *x;
    const float *m;
    const float *ga;  // [n][3] or NULL
    const float *gp;  // [n] or NULL
    int n;
    float eps2;
    int chunk;
    float4 *partial;  // [splits][n] (dL/dx, dL/dm) per split when PARTIAL
    float *gx;
    float *gm;
};

// Row groups with the leap-frog update instead of the stores.
struct BwdEpiArgs : BwdArgs {
    LfEpi e;
};

struct RowAcc {
    float A, Bx, By, Bz, Cx, Cy, Cz, G;
};

__device__ __forceinline__ void adj_term(float xk, float yk, float zk, float mk, float wkx,
                                         float wky, float wkz, float vk, float4 q, float4 wq,
                                         float eps2, bool skip, RowAcc &t)
{
    const float dx = xk - q.x;
    const float dy = yk - q.y;
    const float dz = zk - q.z;
    float s = __builtin_fmaf(dx, dx, eps2);
    s = __builtin_fmaf(dy, dy, s);
    s = __builtin_fmaf(dz, dz, s);
    const float r = skip ? 0.0f : __builtin_amdgcn_rsqf(s);
    const float r2 = r * r;
    const float r3 = r * r2;
    // A += m_j r^3 ; B += r^3 w_j
    t.A = __builtin_fmaf(q.w, r3, t.A);
    t.Bx = __builtin_fmaf(r3, wq.x, t.Bx);
    t.By = __builtin_fmaf(r3, wq.y, t.By);
    t.Bz = __builtin_fmaf(r3, wq.z, t.Bz);
    // c . d = m_j (w_k . d) - m_k (w_j . d)
    float wkd = wkx * dx;
    wkd = __builtin_fmaf(wky, dy, wkd);
    wkd = __builtin_fmaf(wkz, dz, wkd);
    float wjd = wq.x * dx;
    wjd = __builtin_fmaf(wq.y, dy, wjd);
    wjd = __builtin_fmaf(wq.z, dz, wjd);
    const float cd = __builtin_fmaf(q.w, wkd, -mk * wjd);
    // b = m_j v_k + m_k v_j
    const float b = __builtin_fmaf(mk, wq.w, q.w * vk);
    // u = r^3 (3 r^2 (c . d) + b) ; C += u d
    const float u = r3 * __builtin_fmaf(3.0f * r2, cd, b);
    t.Cx = __builtin_fmaf(u, dx, t.Cx);
    t.Cy = __builtin_fmaf(u, dy, t.Cy);
    t.Cz = __builtin_fmaf(u, dz, t.Cz);
    // dL/dm_k += r v_j - r^3 (w_j . d)
    t.G = __builtin_fmaf(r, wq.w, t.G);
    t.G = __builtin_fmaf(-r3, wjd, t.G);
}

__device__ __forceinline__ void fold(RowAcc &acc, const RowAcc &t)
{
    acc.A += t.A;
    acc.Bx += t.Bx;
    acc.By += t.By;
    acc.Bz += t.Bz;
    acc.Cx += t.Cx;
    acc.Cy += t.Cy;
    acc.Cz += t.Cz;
    acc.G += t.G;
}

__device__ __forceinline__ void zero(RowAcc &t) { t.A = t.Bx = t.By = t.Bz = t.Cx = t.Cy = t.Cz = t.G = 0.0f; }

__device__ __forceinline__ float4 load_xm(const BwdArgs &P, int j)
{
    return make_float4(P.x[3 * j], P.x[3 * j + 1], P.x[3 * j + 2], P.m[j]);
}

__device__ __forceinline__ float4 load_wv(const BwdArgs &P, int j)
{
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (P.ga) {
        r.x = P.ga[3 * j];
        r.y = P.ga[3 * j + 1];
        r.z = P.ga[3 * j + 2];
    }
    if (P.gp) r.w = P.gp[j];
    return r;
}

template <int BLOCK, int K, int U, bool PARTIAL>
__global__ __launch_bounds__(BLOCK) void backward_kernel(BwdArgs P)
{
    constexpr int TILE = BLOCK;
    __shared__ float4 tile_xm[TILE];
    __shared__ float4 tile_wv[TILE];

    const int tid = threadIdx.x;
    const int n = P.n;
    const int i0 = blockIdx.x * (BLOCK * K);
    const int jbeg = blockIdx.y * P.chunk;
    const int jend = min(n, jbeg + P.chunk);
    const float eps2 = P.eps2;

    float4 xk[K], wk[K];
    int kk[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = i0 + k * BLOCK + tid;
        kk[k] = i;
        const int ic = i < n ? i : n - 1;
        xk[k] = load_xm(P, ic);
        wk[k] = load_wv(P, ic);
    }
    RowAcc acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) zero(acc[k]);

    float4 nxm = make_float4(0.f, 0.f, 0.f, 0.f), nwv = nxm;
    if (jbeg + tid < jend) {
        nxm = load_xm(P, jbeg + tid);
        nwv = load_wv(P, jbeg + tid);
    }

    const int iblk_end = i0 + BLOCK * K;
    for (int t0 = jbeg; t0 < jend; t0 += TILE) {
        __syncthreads();
        tile_xm[tid] = nxm;
        tile_wv[tid] = nwv;
        __syncthreads();
        {
            const int j = t0 + TILE + tid;
            nxm = make_float4(0.f, 0.f, 0.f, 0.f);
            nwv = nxm;
            if (j < jend) {
                nxm = load_xm(P, j);
                nwv = load_wv(P, j);
            }
        }
        RowAcc t[K];
#pragma unroll
        for (int k = 0; k < K; ++k) zero(t[k]);

        const int cnt = min(TILE, jend - t0);
        const bool masked = (cnt < TILE) || (t0 < iblk_end && t0 + TILE > i0);
        if (!masked) {
            for (int jj = 0; jj < TILE; jj += U) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float4 q = tile_xm[jj + u];
                    const float4 wq = tile_wv[jj + u];
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        adj_term(xk[k].x, xk[k].y, xk[k].z, xk[k].w, wk[k].x, wk[k].y, wk[k].z,
                                 wk[k].w, q, wq, eps2, false, t[k]);
                }
            }
        } else {
            for (int jj = 0; jj < cnt; ++jj) {
                const float4 q = tile_xm[jj];
                const float4 wq = tile_wv[jj];
                const int j = t0 + jj;
#pragma unroll
                for (int k = 0; k < K; ++k)
                    adj_term(xk[k].x, xk[k].y, xk[k].z, xk[k].w, wk[k].x, wk[k].y, wk[k].z,
                             wk[k].w, q, wq, eps2, j == kk[k], t[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) fold(acc[k], t[k]);
    }

#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = kk[k];
        if (i >= n) continue;
        // dL/dx_k = w_k A - m_k B - C
        const RowAcc &c = acc[k];
        const float gx = wk[k].x * c.A - xk[k].w * c.Bx - c.Cx;
        const float gy = wk[k].y * c.A - xk[k].w * c.By - c.Cy;
        const float gz = wk[k].z * c.A - xk[k].w * c.Bz - c.Cz;
        if (PARTIAL) {
            P.partial[(size_t)blockIdx.y * n + i] = make_float4(gx, gy, gz, c.G);
        } else {
            P.gx[3 * i + 0] = gx;
            P.gx[3 * i + 1] = gy;
            P.gx[3 * i + 2] = gz;
            if (P.gm) P.gm[i] = c.G;
        }
    }
}

// Row-group adjoint for small and middle n, as the forward's row groups: a
// workgroup of four waves owns K rows (the same in every lane), wave w meets
// the 64-particle tiles w, w + 4, ... with both its particles (x, m) and
// their weights (w, v) loaded ahead, and gathers the sums A, B, C, G.  Each
// lane combines its own into dL/dx (w A and C are large next to their
// difference where the field is smooth: combined after the sums over the lanes,
// dL/dx of 5,000 bodies in a cube was 3 times as far from float64), and the
// four sums per row are added by shared halvings, then in float64, and over the
// waves in order.  One launch, no partials, bitwise reproducible.  HAS_V false: no
// potential weights, whose terms are not formed (bitwise the result of zero
// weights).
//
// Bound by VALU issue (31 operations per ordered pair, 28 without potential
// weights): 92 cycles per 64 pairs and SIMD at 16,384 bodies with K = 4, about
// 10 of them the loads.  Per call with potential weights, one row per wave
// before: 7.4 -> 6.2 us at 2,000 bodies, 11.8 -> 8.9 at 2,500, 13.4 -> 9.6 at
// 3,000.
constexpr int kBwdRowMax = 4;  // rows per group

// One tile of 64 particles (q, wq of this lane) for K rows, with the opposite
// difference e = x_j - x_k = -d, so that every term below is a plain product
// or accumulating FMA (two-operand encodings; a negated operand would need
// the longer one, which issues slower): with
//     c . e = m_j (w_k . e) + (-m_k) (w_j . e)
//     u = r^3 (3 r^2 (c . e) + b') = -r^3 (3 r^2 (c . d) - b'),  b' = -b
// the sums are A, B, G += r v_j + r^3 (w_j . e) and C += u e
// (u e = r^3 (3 r^2 (c . d) + b) d).  MASKED: lanes whose particle is a row
// itself, or past n, take r = 0.
template <int K, bool HAS_V, bool MASKED>
__device__ __forceinline__ void adj_row_tile(const float4 (&xk)[K], const float4 (&wk)[K],
                                             const float (&mn)[K], float4 q, float4 wq,
                                             float eps2, int j, int i0, int n,
                                             float4 (&bg)[K], float4 (&ca)[K])
{
    float ex[K], ey[K], ez[K], rr[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        ex[k] = q.x - xk[k].x;
        ey[k] = q.y - xk[k].y;
        ez[k] = q.z - xk[k].z;
        float s = __builtin_fmaf(ex[k], ex[k], eps2);
        s = __builtin_fmaf(ey[k], ey[k], s);
        rr[k] = __builtin_fmaf(ez[k], ez[k], s);
    }
    rsq_group<K>(rr);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (MASKED && (j == i0 + k || j >= n)) rr[k] = 0.0f;
        const float r = rr[k];
        const float r2 = r * r;
        const float r3 = r * r2;
        float4 &b = bg[k], &c = ca[k];  // (B, G), (C, A)
        c.w = __builtin_fmaf(q.w, r3, c.w);
        b.x = __builtin_fmaf(r3, wq.x, b.x);
        b.y = __builtin_fmaf(r3, wq.y, b.y);
        b.z = __builtin_fmaf(r3, wq.z, b.z);
        float wke = wk[k].x * ex[k];
        wke = __builtin_fmaf(wk[k].y, ey[k], wke);
        wke = __builtin_fmaf(wk[k].z, ez[k], wke);
        float wje = wq.x * ex[k];
        wje = __builtin_fmaf(wq.y, ey[k], wje);
        wje = __builtin_fmaf(wq.z, ez[k], wje);
        const float ce = __builtin_fmaf(q.w, wke, mn[k] * wje);
        // mn = -m_k, wk.w = -v_k here.  The 3 goes to r^2, whose rounding differs
        // from pair to pair: to the masses, a set of equal ones all rounded alike.
        const float r23 = 3.0f * r2;
        const float e = HAS_V ? __builtin_fmaf(r23, ce, __builtin_fmaf(mn[k], wq.w, q.w * wk[k].w))
                              : r23 * ce;
        const float u = r3 * e;
        c.x = __builtin_fmaf(u, ex[k], c.x);
        c.y = __builtin_fmaf(u, ey[k], c.y);
        c.z = __builtin_fmaf(u, ez[k], c.z);
        if (HAS_V) b.w = __builtin_fmaf(r, wq.w, b.w);
        b.w = __builtin_fmaf(r3, wje, b.w);
    }
}

template <int K, bool HAS_V, bool EPI = false>
__global__ __launch_bounds__(256) void backward_row_kernel(
    typename std::conditional<EPI, BwdEpiArgs, BwdArgs>::type P)
{
    constexpr int D = K <= 2 ? 4 : 2;  // tiles loaded ahead
    __shared__ double red[4][4 * K];
    const int n = P.n;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int i0 = blockIdx.x * K;
    float eps2 = P.eps2;
    in_vgpr(eps2);
    const auto bx = make_buffer(P.x, 12u * (unsigned)n), bm = make_buffer(P.m, 4u * (unsigned)n);
    // an absent weight array is an empty buffer: its loads give zero
    const auto bw = make_buffer(P.ga, P.ga ? 12u * (unsigned)n : 0u);
    const auto bv = make_buffer(P.gp, P.gp ? 4u * (unsigned)n : 0u);
    const auto weights = [&](unsigned j) {
        float4 v = buffer_xm(bw, bv, j);
        if (!HAS_V) v.w = 0.f;
        return v;
    };
    float4 xk[K], wk[K];
    float mn[K];  // -m_k
    float4 bg[K], ca[2][K];  // C and A of every second tile apart: half the chain
#pragma unroll
    for (int k = 0; k < K; ++k) {
        bg[k] = ca[0][k] = ca[1][k] = make_float4(0.f, 0.f, 0.f, 0.f);
        const unsigned ic = (unsigned)min(i0 + k, n - 1);  // rows past n are computed, not stored
        xk[k] = buffer_xm(bx, bm, ic);
        wk[k] = weights(ic);
        wk[k].w = -wk[k].w;
        mn[k] = -xk[k].w;
    }
    const int full = n >> 6;  // tiles without particles past n
    const int self0 = i0 >> 6, self1 = min(i0 + K - 1, n - 1) >> 6;
    float4 q[D], wq[D];
    const auto load = [&](int t, float4 &a, float4 &b) {
        const unsigned j = (unsigned)(t * 64 + lane);
        a = buffer_xm(bx, bm, j);
        b = weights(j);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(wv + 4 * d, q[d], wq[d]);
    const auto masked = [&](int t) {
        float4 a, b;
        load(t, a, b);
        adj_row_tile<K, HAS_V, true>(xk, wk, mn, a, b, eps2, t * 64 + lane, i0, n, bg,
                                      ca[0]);
    };
    // the tiles with pairs to leave out first, as in the forward kernel
    for (int t = self0; t <= self1; ++t)
        if ((t & 3) == wv) masked(t);
    if ((n & 63) != 0 && (full & 3) == wv && full > self1) masked(full);
    for (int t0 = wv; t0 < full; t0 += 4 * D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int t = t0 + 4 * d;
            if (t < full && (t < self0 || t > self1))
                adj_row_tile<K, HAS_V, false>(xk, wk, mn, q[d], wq[d], eps2, 0, 0, 0, bg,
                                               ca[d & 1]);
            load(t + 4 * D, q[d], wq[d]);
        }
    }
    float sums[K][4];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        // dL/dx_k = w_k A - m_k B - C, lane by lane
        float3 d[2];  // w A - C
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const float4 &f = ca[e][k];
            d[e] = make_float3(__builtin_fmaf(wk[k].x, f.w, -f.x), __builtin_fmaf(wk[k].y, f.w, -f.y),
                               __builtin_fmaf(wk[k].z, f.w, -f.z));
        }
        sums[k][0] = __builtin_fmaf(mn[k], bg[k].x, d[0].x + d[1].x);
        sums[k][1] = __builtin_fmaf(mn[k], bg[k].y, d[0].y + d[1].y);
        sums[k][2] = __builtin_fmaf(mn[k], bg[k].z, d[0].z + d[1].z);
        sums[k][3] = bg[k].w;
    }
    wave_sums<K>(sums, lane, [&](int k, double s) { red[wv][4 * k + quad_of_row(lane >> 4)] = s; });
    __syncthreads();
    // thread 4 k + c stores component c of row i0 + k (c == 3: dL/dm)
    const int k = threadIdx.x >> 2, c = threadIdx.x & 3;
    const int i = i0 + k;
    if (k >= K || i >= n) return;
    double sum = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < 4; ++w) sum += red[w][threadIdx.x];
    const float g = (float)sum;
    if (c == 3) {
        if constexpr (EPI)
            P.e.lm[i] = __builtin_fmaf(P.e.c, g, P.e.lm[i]);
        else if (P.gm)
            P.gm[i] = g;
    } else if constexpr (EPI) {
        lf_coord(P.e, 3 * (size_t)i + c, g);
    } else {
        P.gx[3 * (size_t)i + c] = g;
    }
}

using RowFn = void (*)(const BwdArgs &, const LfEpi *, hipStream_t);

template <int K>
static void launch_bwd_rows(const BwdArgs &P, const LfEpi *epi, hipStream_t stream)
{
    const dim3 grid((unsigned)((P.n + K - 1) / K));
    if (epi)
        hipLaunchKernelGGL((backward_row_kernel<K, false, true>), grid, dim3(256), 0, stream,
                           (BwdEpiArgs{P, *epi}));
    else if (P.gp)
        hipLaunchKernelGGL((backward_row_kernel<K, true>), grid, dim3(256), 0, stream, P);
    else
        hipLaunchKernelGGL((backward_row_kernel<K, false>), grid, dim3(256), 0, stream, P);
}

__global__ __launch_bounds__(256) void backward_reduce_kernel(const float4 *__restrict__ partial,
                                                              int splits, int n, float *gx,
                                                              float *gm)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float4 s = partial[i];
    for (int k = 1; k < splits; ++k) {
        const float4 q = partial[(size_t)k * n + i];
        s.x += q.x;
        s.y += q.y;
        s.z += q.z;
        s.w += q.w;
    }
    gx[3 * i + 0] = s.x;
    gx[3 * i + 1] = s.y;
    gx[3 * i + 2] = s.z;
    if (gm) gm[i] = s.w;
}

// ---------------------------------------------------------------------------
// Pair-once adjoint.  With d = x_k - x_j, c_kj = m_j w_k - m_k w_j and
// b_kj = m_j v_k + m_k v_j, the x-gradient term
//     F(k, j) = r^3 c_kj - r^3 (3 r^2 (c_kj . d) + b_kj) d
// satisfies F(j, k) = -F(k, j) (c and d flip sign, b and c.d do not), so one
// evaluation serves both rows: dL/dx_k += F, dL/dx_j -= F.  The mass terms
//     dL/dm_k += r v_j - r^3 (w_j . d),   dL/dm_j += r v_k + r^3 (w_k . d)
// share r, r^3 and the two dot products.  The block/ring decomposition, LDS
// slot read-modify-writes and partial slots are those of the pair-once
// forward kernel (pair_once.hpp), diagonal tiles included; tiles hold two
// float4 per particle.

struct SymBwdArgs {
    const float *x;
    const float *m;
    const float *ga;
    const float *gp;
    int n;
    float eps2;
    int M;
    int C;
    int d_lo, d_hi;   // ring deltas of this launch's group
    float4 *partial;  // [C + G][n]: (dL/dx, dL/dm)
    int held;         // held_tiles of the longest chunk
};

// A lane's row constants in the form the pair terms read (all terms are then
// plain products and accumulating FMAs; a negated operand would take the long
// encoding).
struct AdjRow {
    float x, y, z, m;      // position, mass
    float mn;              // -m
    float wx, wy, wz, v;   // weights
    float vn;              // -v
};

// The first R rows (from row B on, in groups of four) of a lane against the
// tile particle (q, wq), each pair met once, the rows' reciprocal square roots
// as one group.  With e = x_j - x_k = -d:
//     F = r^3 (c - t d) = r^3 (c + t e),  t = 3 r^2 (c . d) + b
//     c . d = m_k (w_j . e) - m_j (w_k . e)
// enters tk as +F and the slot ja as +F too, which the slots' readers negate,
// as the j mass term r v_k + r^3 (w_k . d) = r v_k - r^3 (w_k . e): the slot
// takes its opposite, r^3 (w_k . e) - r v_k.
template <int K, bool HAS_V, int R = K, int B = 0>
__device__ __forceinline__ void adj_pair_rows(const AdjRow (&row)[K], const float4 &q,
                                              const float4 &wq, float qn, float eps2,
                                              float4 (&tk)[K], float4 &ja)
{
    constexpr int G = R < 4 ? R : 4;
    float ex[G], ey[G], ez[G], rr[G];
#pragma unroll
    for (int k = 0; k < G; ++k) {
        ex[k] = q.x - row[B + k].x;
        ey[k] = q.y - row[B + k].y;
        ez[k] = q.z - row[B + k].z;
        float s = __builtin_fmaf(ex[k], ex[k], eps2);
        s = __builtin_fmaf(ey[k], ey[k], s);
        rr[k] = __builtin_fmaf(ez[k], ez[k], s);
    }
    rsq_group<G>(rr);
#pragma unroll
    for (int k = 0; k < G; ++k) {
        const AdjRow &w = row[B + k];
        float4 &t4 = tk[B + k];
        const float r = rr[k];
        const float r2 = r * r;
        const float r3 = r * r2;
        float wke = w.wx * ex[k];
        wke = __builtin_fmaf(w.wy, ey[k], wke);
        wke = __builtin_fmaf(w.wz, ez[k], wke);
        float wje = wq.x * ex[k];
        wje = __builtin_fmaf(wq.y, ey[k], wje);
        wje = __builtin_fmaf(wq.z, ez[k], wje);
        const float cd = __builtin_fmaf(qn, wke, w.m * wje);
        // The 3 goes to r^2, whose rounding differs from pair to pair: to the
        // masses, a set of equal ones all rounded alike (10,600 bodies of one mass
        // in a cube, eps2 0.01: dL/dx 1.2e-7 from float64, 0.7e-7 so).
        // Without potential weights (v = 0) b vanishes and t is exactly the fused
        // form with a zero addend.
        const float r23 = 3.0f * r2;
        const float t = HAS_V ? __builtin_fmaf(r23, cd, __builtin_fmaf(w.m, wq.w, q.w * w.v))
                              : r23 * cd;
        const float ux = __builtin_fmaf(t, ex[k], __builtin_fmaf(q.w, w.wx, w.mn * wq.x));
        const float uy = __builtin_fmaf(t, ey[k], __builtin_fmaf(q.w, w.wy, w.mn * wq.y));
        const float uz = __builtin_fmaf(t, ez[k], __builtin_fmaf(q.w, w.wz, w.mn * wq.z));
        t4.x = __builtin_fmaf(r3, ux, t4.x);
        t4.y = __builtin_fmaf(r3, uy, t4.y);
        t4.z = __builtin_fmaf(r3, uz, t4.z);
        if (HAS_V) t4.w = __builtin_fmaf(r, wq.w, t4.w);
        t4.w = __builtin_fmaf(r3, wje, t4.w);
        ja.x = __builtin_fmaf(r3, ux, ja.x);
        ja.y = __builtin_fmaf(r3, uy, ja.y);
        ja.z = __builtin_fmaf(r3, uz, ja.z);
        ja.w = __builtin_fmaf(r3, wke, ja.w);
        if (HAS_V) ja.w = __builtin_fmaf(r, w.vn, ja.w);
    }
    if constexpr (R > 4) {
        __builtin_amdgcn_sched_barrier(0);
        adj_pair_rows<K, HAS_V, R - 4, B + 4>(row, q, wq, qn, eps2, tk, ja);
    }
}

// The k-side alone, with the pair removed when `skip` holds (diagonal tiles).
__device__ __forceinline__ void adj_row_term(const float4 &xk, const float4 &wk, const float4 &q,
                                             const float4 &wq, float eps2, bool skip, float4 &tk)
{
    const float dx = xk.x - q.x;
    const float dy = xk.y - q.y;
    const float dz = xk.z - q.z;
    float s = __builtin_fmaf(dx, dx, eps2);
    s = __builtin_fmaf(dy, dy, s);
    s = __builtin_fmaf(dz, dz, s);
    const float r = skip ? 0.0f : __builtin_amdgcn_rsqf(s);
    const float r2 = r * r;
    const float r3 = r * r2;
    float wkd = wk.x * dx;
    wkd = __builtin_fmaf(wk.y, dy, wkd);
    wkd = __builtin_fmaf(wk.z, dz, wkd);
    float wjd = wq.x * dx;
    wjd = __builtin_fmaf(wq.y, dy, wjd);
    wjd = __builtin_fmaf(wq.z, dz, wjd);
    const float cd = __builtin_fmaf(q.w, wkd, -xk.w * wjd);
    const float b = __builtin_fmaf(xk.w, wq.w, q.w * wk.w);
    const float t = __builtin_fmaf(3.0f * r2, cd, b);
    tk.x = __builtin_fmaf(r3, __builtin_fmaf(-t, dx, __builtin_fmaf(q.w, wk.x, -xk.w * wq.x)), tk.x);
    tk.y = __builtin_fmaf(r3, __builtin_fmaf(-t, dy, __builtin_fmaf(q.w, wk.y, -xk.w * wq.y)), tk.y);
    tk.z = __builtin_fmaf(r3, __builtin_fmaf(-t, dz, __builtin_fmaf(q.w, wk.z, -xk.w * wq.z)), tk.z);
    tk.w = __builtin_fmaf(r, wq.w, tk.w);
    tk.w = __builtin_fmaf(-r3, wjd, tk.w);
}

constexpr float kBwdPadRow = 1e18f;
constexpr float kBwdPadCol = -1e18f;

__device__ __forceinline__ void load_xw(const SymBwdArgs &A, int j, float4 &xm, float4 &wv)
{
    if (j < A.n) {
        xm = make_float4(A.x[3 * j], A.x[3 * j + 1], A.x[3 * j + 2], A.m[j]);
        wv = make_float4(A.ga ? A.ga[3 * j] : 0.f, A.ga ? A.ga[3 * j + 1] : 0.f,
                         A.ga ? A.ga[3 * j + 2] : 0.f, A.gp ? A.gp[j] : 0.f);
    } else {
        xm = make_float4(kBwdPadCol, kBwdPadCol, kBwdPadCol, 0.f);
        wv = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// acc += tk; tk = 0.
template <int K>
__device__ __forceinline__ void add_rows(float4 (&acc)[K], float4 (&tk)[K])
{
#pragma unroll
    for (int k = 0; k < K; ++k) {
        acc[k].x += tk[k].x;
        acc[k].y += tk[k].y;
        acc[k].z += tk[k].z;
        acc[k].w += tk[k].w;
        tk[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// The steps of diagonal tile t for one wave (lane l meets tile particle
// (l + s) mod 64 at step s): row tile a = a0 + k pair-once if a < t,
// masked ordered pairs if a == t, nothing if a > t (met on diagonal tile a).
template <int K>
__device__ __forceinline__ void adj_diag_steps(const AdjRow (&row)[K], const int (&kk)[K],
                                               const float4 *tile_xm, const float4 *tile_wv,
                                               float4 *slot, int lane, int a0, int t, int jbase,
                                               float eps2, float4 (&tk)[K])
{
    const bool any_once = a0 < t;
    float4 q = tile_xm[lane];
    float4 wq = tile_wv[lane];
    for (int s = 0; s < 64; ++s) {
        const int jj = (lane + s) & 63;
        // keep this step's slot read after the previous step's write
        __asm__ volatile("" ::: "memory");
        float4 ja = make_float4(0.f, 0.f, 0.f, 0.f);
        if (any_once) ja = slot[jj];
        const float4 qn = tile_xm[(jj + 1) & 63];
        const float4 wqn = tile_wv[(jj + 1) & 63];
        const float nq = -q.w;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (a0 + k < t) {
                const AdjRow one[1] = {row[k]};
                float4 tk1[1] = {tk[k]};
                adj_pair_rows<1, true>(one, q, wq, nq, eps2, tk1, ja);
                tk[k] = tk1[0];
            } else if (a0 + k == t) {
                const AdjRow &w = row[k];
                adj_row_term(make_float4(w.x, w.y, w.z, w.m), make_float4(w.wx, w.wy, w.wz, w.v), q,
                             wq, eps2, jbase + jj == kk[k], tk[k]);
            }
        }
        if (any_once) slot[jj] = ja;
        q = qn;
        wq = wqn;
    }
}

// Ring tiles: the tiles are staged twice (entries e and e + 64 hold
// particle e) and the wave's j-side slots number 128, so lane l at step s
// reads entry l + s and updates slot l + s with no index wrap (immediate
// LDS offsets in the unrolled loop); particle e's j-side sum is slot e plus
// slot e + 64.  Same scheme and ordering argument as the forward pair-once
// kernel.
//
// The slots are emptied every kAdjSlotSteps steps into the lane's sum of its tile
// particle, which ends in its slot, and one-wave blocks add their row sums tk to
// acc in the middle of the tile: a slot's float32 chain grows with the rows per
// lane, and a tile has one wave where two shared its steps before.  Error of
// dL/dm against float64 (2-norm) at 16,384 bodies: two rows per lane and one
// chain per tile 2.4e-7, four rows 2.9e-7, four rows so 1.9e-7 (emptied every 16
// steps 2.1e-7: at 10,600 bodies 4% above the two waves' sums).  Calls take 1%
// longer.
template <int W, int K>
constexpr int kAdjSlotSteps = W == 1 && K == 4 ? 8 : 16;

template <int W, int K, bool HAS_V = true>
__device__ __forceinline__ void adj_ring_steps(const AdjRow (&row)[K], const float4 *tile_xm,
                                               const float4 *tile_wv, float4 *slot, int lane,
                                               float eps2, float4 (&tk)[K], float4 (&acc)[K])
{
    constexpr int kSteps = kAdjSlotSteps<W, K>;
    const float4 *txm = tile_xm + lane;
    const float4 *twv = tile_wv + lane;
    float4 *sl = slot + lane;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 q = txm[0], wq = twv[0], sum = zero;
#pragma nounroll
    for (int h = 0; h < 64 / kSteps; ++h) {
#pragma unroll 4
        for (int s = 0; s < kSteps; ++s) {
            // keep this step's slot read after the previous step's write
            __asm__ volatile("" ::: "memory");
            float4 ja = sl[s];
            const float4 qn = txm[s + 1];
            const float4 wqn = twv[s + 1];
            adj_pair_rows<K, HAS_V>(row, q, wq, -q.w, eps2, tk, ja);
            sl[s] = ja;
            q = qn;
            wq = wqn;
        }
        txm += kSteps;
        twv += kSteps;
        sl += kSteps;
        __asm__ volatile("" ::: "memory");
        const float4 lo = slot[lane];
        const float4 hi = slot[lane + 64];
        sum.x += lo.x + hi.x;
        sum.y += lo.y + hi.y;
        sum.z += lo.z + hi.z;
        sum.w += lo.w + hi.w;
        slot[lane] = zero;
        slot[lane + 64] = zero;
        if (W == 1 && h == 32 / kSteps - 1) add_rows(acc, tk);
    }
    __asm__ volatile("" ::: "memory");
    slot[lane] = sum;
}

// One step s of a one-wave block's diagonal tile: rows k < R meet entry l + s
// pair-once.
template <int K, int R, bool HAS_V>
__device__ __forceinline__ void adj_diag_step(const AdjRow (&row)[K], const float4 *txm,
                                              const float4 *twv, float4 *sl, int s, float eps2,
                                              float4 (&tk)[K])
{
    if constexpr (R > 0) {
        // keep this step's slot read after the previous step's write
        __asm__ volatile("" ::: "memory");
        const float4 q = txm[s];
        const float4 wq = twv[s];
        float4 ja = sl[s];
        adj_pair_rows<K, HAS_V, R>(row, q, wq, -q.w, eps2, tk, ja);
        sl[s] = ja;
    }
}

// Diagonal tile t of a one-wave block, whose rows are the wave's row group t:
// row groups k < t meet it pair-once, and group t its own 64 particles (lane l
// and particle l + s for s = 1..31; at s = 32 both lanes of a pair take their
// own side), as diag_self_steps of the forward.  Loops of two steps kept rolled:
// there are K instances.  Calls against masked ordered pairs, one row at a
// time, with / without potential weights: 37.0 / 34.9 -> 35.8 / 33.9 us at 8,000
// bodies, 48.1 -> 43.8 at 9,000, 74.7 / 70.8 -> 74.0 / 67.5 at 12,500, 123.6 /
// 114.2 -> 122.9 / 111.6 at 16,384, 612 / 561 -> 613 / 549 at 39,000.
template <int K, bool HAS_V, int KT = 0>
__device__ __forceinline__ void adj_self_steps(int t, const AdjRow (&row)[K], const float4 *tile_xm,
                                               const float4 *tile_wv, float4 *slot, int lane,
                                               float eps2, float4 (&tk)[K])
{
    if (t != KT) {
        if constexpr (KT + 1 < K)
            adj_self_steps<K, HAS_V, KT + 1>(t, row, tile_xm, tile_wv, slot, lane, eps2, tk);
        return;
    }
    const float4 *txm = tile_xm + lane;
    const float4 *twv = tile_wv + lane;
    float4 *sl = slot + lane;
    adj_diag_step<K, KT, HAS_V>(row, txm, twv, sl, 0, eps2, tk);
#pragma nounroll
    for (int s = 1; s < 31; s += 2) {
        adj_diag_step<K, KT + 1, HAS_V>(row, txm, twv, sl, s, eps2, tk);
        adj_diag_step<K, KT + 1, HAS_V>(row, txm, twv, sl, s + 1, eps2, tk);
    }
    adj_diag_step<K, KT + 1, HAS_V>(row, txm, twv, sl, 31, eps2, tk);
    adj_diag_step<K, KT, HAS_V>(row, txm, twv, sl, 32, eps2, tk);
    const AdjRow &w = row[KT];
    adj_row_term(make_float4(w.x, w.y, w.z, w.m), make_float4(w.wx, w.wy, w.wz, w.v), txm[32],
                 twv[32], eps2, false, tk[KT]);
    if (KT > 0) {
#pragma nounroll
        for (int s = 33; s < 63; s += 2) {
            adj_diag_step<K, KT, HAS_V>(row, txm, twv, sl, s, eps2, tk);
            adj_diag_step<K, KT, HAS_V>(row, txm, twv, sl, s + 1, eps2, tk);
        }
        adj_diag_step<K, KT, HAS_V>(row, txm, twv, sl, 63, eps2, tk);
    }
    __asm__ volatile("" ::: "memory");
    const float4 lo = slot[lane];
    const float4 hi = slot[lane + 64];
    slot[lane] = make_float4(lo.x + hi.x, lo.y + hi.y, lo.z + hi.z, lo.w + hi.w);
}

// HAS_V false: no potential weights (grad_p NULL); their terms are not
// formed on ring tiles (bitwise the same result as v = 0).
// Each wave owns K * 64 of the block's rows.  Buffers, barriers, slot sums and the tile split of one-wave blocks (T waves)
// as in pair_once_block.
template <int W>
constexpr int kAdjSplit = W == 1 ? kTileSplit : 1;
template <int W>
constexpr int kAdjThreads = 64 * W * kAdjSplit<W>;

template <int W, int K, bool HAS_V, bool HELD = W != 1>
__global__ __launch_bounds__(kAdjThreads<W>, W == 1 && K == 4 ? 3 : 1) void backward_sym_kernel(SymBwdArgs A)
{
    constexpr int PB = W * 64 * K;
    constexpr int TPB = PB / 64;
    constexpr int NB = kSymBuffers<W>;
    constexpr int T = kAdjSplit<W>;
    static_assert(K * 64 <= kTileLds + kTileLds + kSlotLds, "row sums fit a wave's region");
    // per set of W waves: the tile twice over, its weights, the W slot arrays
    constexpr int kLds = NB * (2 * kTileLds + W * kSlotLds);
    __shared__ float4 lds[T * kLds];

    const int lane = threadIdx.x & 63;
    const int tw = T > 1 ? (int)(threadIdx.x >> 6) : 0;  // which of T sub-chunks
    const int tid = T > 1 ? lane : (int)threadIdx.x;     // thread of the block's W waves
    const int wv = tid >> 6;
    float4 *const tile_xm = lds + tw * kLds;
    float4 *const tile_wv = tile_xm + NB * kTileLds;
    float4(*const jacc)[kSlotLds] = reinterpret_cast<float4(*)[kSlotLds]>(tile_wv + NB * kTileLds);
    const auto block_sync = [&]() {
        if (W == 1)
            __asm__ volatile("" ::: "memory");
        else
            __syncthreads();
    };
    const int n = A.n;
    const int M = A.M, C = A.C;
    const int c = blockIdx.x / M;  // chunk-major (chunk_begin)
    const int I = blockIdx.x - c * M;
    float eps2 = A.eps2;
    in_vgpr(eps2);

    AdjRow row[K];
    float4 acc[K];
    int kk[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int i = I * PB + wv * 64 * K + k * 64 + lane;
        kk[k] = i;
        float4 xm = make_float4(kBwdPadRow, kBwdPadRow, kBwdPadRow, 0.f);
        float4 wv4 = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i < n) load_xw(A, i, xm, wv4);
        row[k] = AdjRow{xm.x, xm.y, xm.z, xm.w, -xm.w, wv4.x, wv4.y, wv4.z, wv4.w, -wv4.w};
        acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    }

    // this chunk's share of the block's tiles in the launch's ring group
    // (diagonal first, then the ring delta-major); all-padding tiles are
    // skipped (uniform)
    const int d_lo = A.d_lo;
    const int dj = group_first_delta(d_lo);
    const int U = group_tiles(I, M, d_lo, A.d_hi, TPB);
    const int u0 = chunk_begin(U, C * T, c * T + tw);
    const int u1 = chunk_begin(U, C * T, c * T + tw + 1);
    int u = u0, delta = 0, jbase = 0;
    for (; u < u1; ++u)
        if ((jbase = tile_base<PB>(u, I, M, d_lo, delta)) < n) break;
    float4 nxm = make_float4(0.f, 0.f, 0.f, 0.f), nwv = nxm;
    if (u < u1 && tid < 64) load_xw(A, jbase + tid, nxm, nwv);
    // the rows have arrived here, so that no wait for them in the tile loop
    // also waits for the prefetch
#pragma unroll
    for (int k = 0; k < K; ++k)
        __asm__ volatile("" : "+v"(row[k].x), "+v"(row[k].y), "+v"(row[k].z), "+v"(row[k].m),
                         "+v"(row[k].wx), "+v"(row[k].wy), "+v"(row[k].wz), "+v"(row[k].v));

    const auto stage = [&](int b) {
        if (tid < 64) {
            tile_xm[b * kTileLds + tid] = nxm;
            tile_wv[b * kTileLds + tid] = nwv;
            tile_xm[b * kTileLds + tid + 64] = nxm;
            tile_wv[b * kTileLds + tid + 64] = nwv;
        }
    };
    const auto clear_slots = [&](int b) {
        jacc[b * W + wv][lane] = make_float4(0.f, 0.f, 0.f, 0.f);
        jacc[b * W + wv][lane + 64] = make_float4(0.f, 0.f, 0.f, 0.f);
    };
    // as in pair_once_block
    [[maybe_unused]] int held = 0;
    bool fresh = true;
    const auto hand_over = [&]() {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (kk[k] < n) {
                float4 *out = A.partial + (size_t)c * n + kk[k];
                float4 v = acc[k];
                if (!fresh) {
                    const float4 w = *out;
                    v = make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
                }
                *out = v;
            }
            acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        held = 0;
        fresh = false;
    };

    int b = 0;
    if (NB == 2 && u < u1) {
        stage(0);
        clear_slots(0);
        __syncthreads();
    }
    while (u < u1) {
        if (NB == 1) {
            block_sync();  // the previous tile and its slot sums are done
            stage(0);
            clear_slots(0);
            block_sync();
        }
        const int cur_u = u, cur_delta = delta, cur_base = jbase;
        for (++u; u < u1; ++u)
            if ((jbase = tile_base<PB>(u, I, M, d_lo, delta)) < n) break;
        if (u < u1 && tid < 64) load_xw(A, jbase + tid, nxm, nwv);

        float4 tk[K];
#pragma unroll
        for (int k = 0; k < K; ++k) tk[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        float4 *slot = &jacc[b * W + wv][0];
        const float4 *txm = tile_xm + b * kTileLds, *twv = tile_wv + b * kTileLds;
        const bool diag = (cur_delta == 0);
        if (!diag)
            adj_ring_steps<W, K, HAS_V>(row, txm, twv, slot, lane, eps2, tk, acc);
        else if constexpr (W == 1)
            adj_self_steps<K, HAS_V>(cur_u, row, txm, twv, slot, lane, eps2, tk);
        else
            adj_diag_steps<K>(row, kk, txm, twv, slot, lane, wv * K, cur_u, cur_base, eps2, tk);
        __asm__ volatile("" ::: "memory");
        add_rows(acc, tk);
        if (NB == 2 && u < u1) stage(b ^ 1);
        block_sync();  // every wave's j-side slots are complete
        if (NB == 2 && u < u1) clear_slots(b ^ 1);
        // every wave left the opposite of particle e's sums in its slot e;
        // they are added in wave order
        if (!diag) {
            float4 *out = A.partial + (size_t)(C + cur_delta - dj) * n + cur_base;
            if constexpr (W == 1) {
                const float4 sum = jacc[0][tid];
                if (cur_base + tid < n) out[tid] = make_float4(-sum.x, -sum.y, -sum.z, -sum.w);
            } else {
                for (int f = tid; f < 256; f += W * 64) {
                    float sum = reinterpret_cast<const float *>(jacc[b * W])[f];
#pragma unroll
                    for (int w2 = 1; w2 < W; ++w2)
                        sum += reinterpret_cast<const float *>(jacc[b * W + w2])[f];
                    if (cur_base + (f >> 2) < n) reinterpret_cast<float *>(out)[f] = -sum;
                }
            }
        } else if (wv == cur_u / K) {
            // this wave holds diagonal tile cur_u's rows (lane-slot cur_u % K);
            // tile particle e's sums are in slot e
            float4 sum = jacc[b * W][lane];
#pragma unroll
            for (int w2 = 1; w2 < W; ++w2) {
                const float4 v = jacc[b * W + w2][lane];
                sum.x += v.x;
                sum.y += v.y;
                sum.z += v.z;
                sum.w += v.w;
            }
            const int kt = cur_u - wv * K;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (k == kt) {
                    acc[k].x -= sum.x;
                    acc[k].y -= sum.y;
                    acc[k].z -= sum.z;
                    acc[k].w -= sum.w;
                }
        }
        if (NB == 2) b ^= 1;
        if (HELD && ++held == A.held) hand_over();
    }
    if constexpr (T == 1) {
        hand_over();
    } else {
        // the T waves' row sums through their own LDS regions
        __asm__ volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < K; ++k) tile_xm[k * 64 + lane] = acc[k];
        __syncthreads();
        float *out = reinterpret_cast<float *>(A.partial + (size_t)c * n + I * PB);
        const float *all = reinterpret_cast<const float *>(lds);
        for (int f = threadIdx.x; f < K * 256; f += T * 64) {
            double sum = all[f];
#pragma unroll
            for (int w = 1; w < T; ++w) sum += all[w * kLds * 4 + f];
            if (I * PB + (f >> 2) < n) out[f] = (float)sum;
        }
    }
}

// Workgroups of W waves per CU (counting each wave of a tile split as one).
template <int W, int K>
nbody_status adj_occupancy(int *per_cu)
{
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        per_cu, backward_sym_kernel<W, K, true>, kAdjThreads<W>, 0);
    if (e != hipSuccess) return hip_fail(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    if (*per_cu < 1) *per_cu = 1;
    *per_cu *= kAdjSplit<W>;
    return NBODY_OK;
}

// The two-row one-wave kernel counted in workgroups of two waves.
nbody_status adj_occupancy_half(int *per_cu)
{
    const nbody_status st = adj_occupancy<1, 2>(per_cu);
    if (st == NBODY_OK) *per_cu = (*per_cu + 1) / 2;
    return st;
}

// Sizes at which the bwd_sym_s2 variants run the row-group kernel instead (as
// kRowBandEnd of the forward).  Whole calls with / without potential weights,
// pair-once (1 x 2, a tile per wave) against row groups: 20.9 / 20.4 and 20.5 / 18.3
// us at 5,000 bodies, 28.0 / 26.4 and 27.1 / 24.5 at 6,001, 28.6 / 27.0 and 31.1 /
// 28.1 at 6,200, 28.9 / 27.2 and 33.0 / 29.7 at 6,500.
constexpr int kBwdRowBandBegin = 4000, kBwdRowBandEnd = 6200;
bool bwd_row_band(int n) { return n >= kBwdRowBandBegin && n < kBwdRowBandEnd; }

const RowFn kRowLaunch[kBwdRowMax + 1] = {nullptr, launch_bwd_rows<1>, launch_bwd_rows<2>,
                                          launch_bwd_rows<3>, launch_bwd_rows<4>};

nbody_status backward_rows_run(int least, const char *name, const Device &dev, const float *x,
                               const float *m, int n, float eps2, const float *ga, const float *gp,
                               float *gx, float *gm, hipStream_t stream, const LfEpi *epi,
                               bool *fused)
{
    const BwdArgs P{x, m, ga, gp, n, eps2, 0, nullptr, gx, gm};
    // an update that changes lv, the weights the other groups still read,
    // needs a second buffer for it
    if (epi && (gp || epi->mode != kLfAdjoint || (epi->chain && !epi->lvo))) epi = nullptr;
    if (epi && fused) *fused = true;
    if (fault_injected("launch")) return fail(NBODY_ERROR_LAUNCH_FAILED, "injected launch fault");
    prof_mark(stream, 0);
    kRowLaunch[row_group_rows(n, dev.num_cu, least, kBwdRowMax, 10)](P, epi, stream);
    prof_mark(stream, 1);
    return check_launch(name);
}

// The launches of a plan whose blocks are KW waves x KK rows.
template <int W, int K, bool HELD = W != 1>
nbody_status launch_backward_sym(const SymPlan &pl, void *ws, const char *name, const float *x,
                                 const float *m, int n, float eps2, const float *ga,
                                 const float *gp, float *gx, float *gm, hipStream_t stream,
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
        SymBwdArgs A{x, m, ga, gp, n, eps2, pl.M, C, 0, 0, partial, held};
        sym_group(pl, g, &A.d_lo, &A.d_hi);
        prof_mark(stream, 0);
        if (gp)
            hipLaunchKernelGGL((backward_sym_kernel<W, K, true, HELD>), dim3(pl.M * C),
                               dim3(kAdjThreads<W>), 0, stream, A);
        else
            hipLaunchKernelGGL((backward_sym_kernel<W, K, false, HELD>), dim3(pl.M * C),
                               dim3(kAdjThreads<W>), 0, stream, A);
        prof_mark(stream, 1);
        nbody_status st = check_launch(name);
        if (st != NBODY_OK) return st;
        const int first = g == 0, last = g == pl.groups - 1;
        if (last && lf)
            hipLaunchKernelGGL((slot_fold_kernel<PB, true>), dim3((n + 63) / 64), dim3(256), 0,
                               stream, partial, n, pl.M, C, A.d_lo, A.d_hi, first, last, acc, gx,
                               gm, *epi);
        else
            hipLaunchKernelGGL((slot_fold_kernel<PB>), dim3((n + 63) / 64), dim3(256), 0, stream,
                               partial, n, pl.M, C, A.d_lo, A.d_hi, first, last, acc, gx, gm,
                               LfEpi{});
        st = check_launch("slot_fold");
        if (st != NBODY_OK) return st;
    }
    if (lf && fused) *fused = true;
    return NBODY_OK;
}

// OCC divides the chunk count and ROUNDS multiplies it (as in the
// pair-once forward kernel).  The kernel may hold a block of W waves x K rows
// as KW waves x KK rows (the same particles and plan); SMALL variants (one
// wave, two rows) run the row-group kernel in its band.
//
// One-wave two-row variants take a tile per wave up to kOneTileEnd, four rows
// per lane (half the LDS traffic per pair, half the slots to fold) from
// kOneTileBegin.  Calls with potential weights, two rows / four rows, a tile per
// wave: 36.0 / 45.4 us at 8,000 bodies, 56.7 / 60.7 at 10,000, 63.7 / 61.9 at
// 11,000; before the slots were emptied within a tile (1-2% less each) 182 / 175
// at 20,000, 394 / 371 at 30,000, 655 / 618 at 39,000, with chunks of one or two
// tiles as planned 40.2 us at 8,000, 182 at 20,000, 660 at 39,000.  Four rows, a
// tile per wave / 2 x 4 (the 4-wave blocks), with and without potential weights:
// 644 / 646 and 580 / 602 us at 40,000, 802 / 792 and 722 / 733 at 45,000, 1032 /
// 976 and 951 / 901 at 50,021.
template <int W, int K, int OCC, int ROUNDS = 1, int KW = W, int KK = K, bool SMALL = false>
nbody_status run_backward_sym(const char *name, const Device &dev, const float *x, const float *m,
                              int n, float eps2, const float *ga, const float *gp, float *gx,
                              float *gm, hipStream_t stream, const LfEpi *epi, bool *fused,
                              const Arena &arena)
{
    static_assert(KW * KK == W * K, "the same block");
    constexpr int PB = W * 64 * K;
    if constexpr (SMALL) {
        if (bwd_row_band(n)) {
            const nbody_status st = rows_for_plan(name, dev, n, stream, arena);
            return st != NBODY_OK ? st
                                  : backward_rows_run(1, name, dev, x, m, n, eps2, ga, gp, gx, gm,
                                                      stream, epi, fused);
        }
    }
    int per_cu = 0;
    nbody_status st = SMALL ? adj_occupancy_half(&per_cu) : adj_occupancy<W, K>(&per_cu);
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
    if constexpr (KW == 1 && KK == 2) {
        SymPlan one;
        if (n >= kOneTileBegin && n < kOneTileEnd && one_tile_plan(n, 4, pl, &one))
            return launch_backward_sym<1, 4>(one, ws, name, x, m, n, eps2, ga, gp, gx, gm, stream,
                                             epi, fused);
        if (n < kOneTileBegin && one_tile_plan(n, 2, pl, &one))
            return launch_backward_sym<1, 2>(one, ws, name, x, m, n, eps2, ga, gp, gx, gm, stream,
                                             epi, fused);
    }
    if (KW == 1) pl.C = (pl.C + kTileSplit - 1) / kTileSplit;  // counted in workgroups
    // Two-wave blocks of 512 keep at most 52 chunks (partials to write and fold per
    // row).  As planned / 76 / 52 / 44 (before the slots were emptied within a tile:
    // 1-2% less each): 647 / 641 / 633 / 640 us at 40,000 bodies (104 planned), 867 /
    // 858 / 845 / 849 at 47,000, 975 / 971 / 959 / 959 at 50,021, 1616 / 1611 / 1604 /
    // 1607 at 65,536.
    if constexpr (KW == 2 && KK == 4 && ROUNDS > 1) {
        if (pl.C > 52) pl.C = 52;
        // short chunks (up to some 90,000 bodies) hand nothing over in between
        if (longest_chunk(pl, KW * KK) <= kHeldTiles)
            return launch_backward_sym<KW, KK, false>(pl, ws, name, x, m, n, eps2, ga, gp, gx, gm,
                                                      stream, epi, fused);
    }
    return launch_backward_sym<KW, KK>(pl, ws, name, x, m, n, eps2, ga, gp, gx, gm, stream, epi,
                                       fused);
}

using KernelFn = void (*)(BwdArgs);

using SymRunFn = nbody_status (*)(const char *, const Device &, const float *, const float *,
                                  int, float, const float *, const float *, float *, float *,
                                  hipStream_t, const LfEpi *, bool *, const Arena &);

// A gather variant (rows own all j) or, with sym set, a pair-once variant
// with W waves, K rows per lane and chunk divisor O.
struct Variant {
    const char *name;
    int block, k, unroll;
    KernelFn direct, partial;
    SymRunFn sym;
    nbody_status (*sym_occupancy)(int *);
    int sym_w, sym_k, sym_occ, sym_rounds;
    bool row;      // row-group kernel, groups of a multiple of row_k rows
    int row_k;
    bool sym_small;  // row groups in bwd_row_band
};

// Particles per pair-once block of a variant.
int sym_block(const Variant &V)
{
    return V.sym_w * 64 * V.sym_k;
}

#define BWD_VARIANT(B, K, U) \
    {"bwd_b" #B "_k" #K "_u" #U, B, K, U, backward_kernel<B, K, U, false>, backward_kernel<B, K, U, true>, nullptr, nullptr, 0, 0, 0, 1}
#define BWD_SYM_VARIANT(W, K, O) \
    {"bwd_sym_w" #W "_k" #K "_o" #O, 0, 0, 0, nullptr, nullptr, run_backward_sym<W, K, O>, \
     adj_occupancy<W, K>, W, K, O, 1}
// Pair-once blocks in R rounds of workgroups (R times the chunks).
#define BWD_SYM_R_VARIANT(W, K, R) \
    {"bwd_sym_w" #W "_k" #K "_r" #R, 0, 0, 0, nullptr, nullptr, run_backward_sym<W, K, 1, R>, \
     adj_occupancy<W, K>, W, K, 1, R}

// The same with each block held by half the waves, twice the rows per lane:
// half the LDS traffic per pair.  GPU time per call with / without potential
// weights, 4 x 2 as 2 x 4: 671 / 612 -> 656 / 596 us at 40,000 bodies, 1016 /
// 932 -> 982 / 898 at 50,021; 8 x 2 as 4 x 4: 27.9 / 25.7 -> 26.4 / 24.0 ms at
// 2^18.
#define BWD_SYM_R_HALF_VARIANT(W, K, R) \
    {"bwd_sym_w" #W "_k" #K "_r" #R, 0, 0, 0, nullptr, nullptr, \
     run_backward_sym<W, K, 1, R, W / 2, 2 * K>, adj_occupancy<W, K>, W, K, 1, R}

// Blocks of 128 rows in plans for workgroups of two waves (half as many chunks
// as the one-wave variants'), R rounds; the row-group kernel in its band.
#define BWD_SYM_S_VARIANT(R) \
    {"bwd_sym_s2_k2_r" #R, 0, 0, 0, nullptr, nullptr, run_backward_sym<1, 2, 1, R, 1, 2, true>, \
     adj_occupancy_half, 1, 2, 1, R, false, 0, true}

#define BWD_ROW_VARIANT(K) \
    {"bwd_row_k" #K, 64, K, 0, nullptr, nullptr, nullptr, nullptr, 0, 0, 0, 1, true, K}

const Variant kVariants[] = {
    BWD_VARIANT(256, 2, 4),
    BWD_VARIANT(256, 1, 8),
    BWD_VARIANT(128, 1, 8),
    BWD_VARIANT(64, 1, 4),
    BWD_VARIANT(64, 1, 8),
    BWD_VARIANT(64, 2, 4),
    BWD_SYM_VARIANT(8, 2, 1),
    BWD_SYM_VARIANT(8, 2, 2),
    BWD_SYM_VARIANT(4, 2, 1),
    BWD_SYM_VARIANT(4, 2, 2),
    BWD_SYM_VARIANT(8, 4, 1),
    BWD_SYM_VARIANT(16, 2, 1),
    BWD_SYM_VARIANT(4, 1, 1),
    BWD_SYM_VARIANT(2, 2, 1),
    BWD_SYM_VARIANT(2, 4, 1),
    BWD_SYM_VARIANT(1, 2, 1),
    BWD_SYM_VARIANT(2, 1, 1),
    BWD_SYM_VARIANT(1, 4, 1),
    BWD_SYM_R_VARIANT(1, 2, 8),
    BWD_SYM_R_VARIANT(2, 2, 8),
    BWD_SYM_R_VARIANT(2, 1, 8),
    BWD_SYM_R_HALF_VARIANT(8, 2, 8),
    BWD_SYM_R_HALF_VARIANT(4, 2, 8),
    BWD_ROW_VARIANT(1),
    BWD_ROW_VARIANT(2),
    BWD_SYM_S_VARIANT(8),
    BWD_SYM_S_VARIANT(16),
    BWD_SYM_R_VARIANT(1, 2, 16),
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

}  // namespace

int backward_variant_count() { return kNumVariants; }

const char *backward_variant_name(int index)
{
    return (index >= 0 && index < kNumVariants) ? kVariants[index].name : nullptr;
}

static int variant_index(const char *name)
{
    for (int v = 0; v < kNumVariants; ++v)
        if (std::strcmp(kVariants[v].name, name) == 0) return v;
    return 0;
}

// Measured on MI355X: the pair-once adjoint wins from about 6,200 particles
// on, row groups below; its workspace is bounded as the forward's (ring
// groups), and above 2^24 particles the gather kernel takes over.  The same
// choice serves calls with and without potential weights.
int backward_default_variant(int64_t n)
{
    static const int pair_once_big = variant_index("bwd_sym_w8_k2_r8");
    static const int pair_once_large = variant_index("bwd_sym_w4_k2_r8");
    static const int pair_once_r8 = variant_index("bwd_sym_w1_k2_r8");
    static const int pair_once_r16 = variant_index("bwd_sym_w1_k2_r16");
    static const int pair_once_small = variant_index("bwd_sym_s2_k2_r8");
    static const int gather = variant_index("bwd_b256_k1_u8");
    static const int row_1 = variant_index("bwd_row_k1");
    static const int row_2 = variant_index("bwd_row_k2");
    if (n > (1 << 24)) return gather;
    // Row groups below 6,200 bodies, then one-wave blocks with a tile per wave
    // up to 40,000: the three variants of that range differ in the plan whose
    // workspace they keep, not in the kernel (run_backward_sym).  Then 4-wave
    // blocks in eight rounds of workgroups (the dispatcher hands short chunks
    // out as slots free up: 10-13% ahead of one round of two-wave blocks with
    // potential weights at 49,152 and 60,000, 9-11% of 8-wave ones at 2^17)
    // and 8-wave blocks from 2^18 (3-7% ahead of one round of them at 2^18
    // and 2^19).  A tile per wave against the 4-wave blocks: run_backward_sym.
    if (n >= (1 << 18)) return pair_once_big;
    if (n >= 40000) return pair_once_large;
    if (n >= 24000 && n < 30000) return pair_once_r16;
    if (n >= 12000) return pair_once_r8;
    if (n >= 4000) return pair_once_small;
    // row groups below 4,000 bodies (an even number of rows from 3,500), which
    // also serve the variant above below kBwdRowBandEnd
    return n >= 3500 ? row_2 : row_1;
}

bool backward_takes_rows(int variant, int n)
{
    const Variant &V = kVariants[variant];
    return V.row || (V.sym_small && bwd_row_band(n));
}

// Geometry of the row gather: j-splits and j per split.
static void bwd_gather_geometry(const Variant &V, int n, int num_cu, int *splits_out,
                                int *chunk_out)
{
    const int iblk = V.block * V.k;
    const int iblocks = (n + iblk - 1) / iblk;
    const int target = 4 * num_cu;
    const int max_splits = (n + V.block - 1) / V.block;
    int splits = (target + iblocks - 1) / iblocks;
    splits = splits < 1 ? 1 : (splits > max_splits ? max_splits : splits);
    int chunk = (n + splits - 1) / splits;
    chunk = (chunk + V.block - 1) / V.block * V.block;
    *splits_out = (n + chunk - 1) / chunk;
    *chunk_out = chunk;
}

int64_t backward_plan_bytes(int variant, int64_t n, int num_cu, int per_cu)
{
    if (variant < 0 || variant >= kNumVariants || n < 0 || n > NBODY_MAX_N || num_cu < 1 ||
        per_cu < 1)
        return -1;
    if (n == 0) return 0;
    const Variant &V = kVariants[variant];
    if (V.row) return 0;
    if (V.sym_small && bwd_row_band((int)n)) return rows_refused(n, sym_workspace_budget(n)) ? -1 : 0;
    if (V.sym) {
        SymPlan pl;
        if (!sym_plan(n, sym_block(V), (int64_t)per_cu * num_cu * V.sym_rounds, V.sym_occ,
                      sym_workspace_budget(n), &pl))
            return -1;
        return (int64_t)pl.bytes();
    }
    int splits = 1, chunk = 0;
    bwd_gather_geometry(V, (int)n, num_cu, &splits, &chunk);
    return splits > 1 ? (int64_t)sizeof(float4) * splits * n : 0;
}

bool backward_alias(int variant, int64_t n, int num_cu, int per_cu)
{
    const int d = backward_default_variant(n);
    const Variant &V = kVariants[variant], &D = kVariants[d];
    if (n <= NBODY_MAX_N && backward_takes_rows(variant, (int)n) && backward_takes_rows(d, (int)n))
        return n < kRowAliasBegin ? !V.row : variant != d;
    // one-tile plans (run_backward_sym) of both
    const auto two_row = [](const Variant &v) { return v.sym && v.sym_w == 1 && v.sym_k == 2; };
    if (variant == d || !two_row(V) || !two_row(D) || n >= kOneTileEnd) return false;
    SymPlan pl, one;
    return sym_plan(n, sym_block(V), (int64_t)per_cu * num_cu * V.sym_rounds, V.sym_occ,
                    sym_workspace_budget(n), &pl) &&
           one_tile_plan(n, n >= kOneTileBegin ? 4 : 2, pl, &one);
}

int64_t backward_variant_max_n(int variant)
{
    if (variant < 0 || variant >= kNumVariants) return -1;
    // the row-group kernels are built for small sizes
    return kVariants[variant].row ? (1 << 16) : NBODY_MAX_N;
}

nbody_status backward_variant_occupancy(int variant, int *per_cu)
{
    const Variant &V = kVariants[variant];
    if (V.sym) return V.sym_occupancy(per_cu);
    const hipError_t e =
        V.row ? hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, backward_row_kernel<kBwdRowMax, true>, 256, 0)
                : hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, V.partial, V.block, 0);
    if (e != hipSuccess) return hip_fail(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    if (*per_cu < 1) *per_cu = 1;
    return NBODY_OK;
}

nbody_status backward_run(int variant, const Device &dev, const float *x, const float *m, int n,
                          float eps2, const float *ga, const float *gp, float *gx, float *gm,
                          hipStream_t stream, const LfEpi *epi, bool *fused, const Arena &arena)
{
    const Variant &V = kVariants[variant];
    if (fused) *fused = false;
    if (V.sym) return V.sym(V.name, dev, x, m, n, eps2, ga, gp, gx, gm, stream, epi, fused, arena);
    if (V.row)
        return backward_rows_run(V.row_k, V.name, dev, x, m, n, eps2, ga, gp, gx, gm, stream, epi,
                                 fused);
    const int iblk = V.block * V.k;
    const int iblocks = (n + iblk - 1) / iblk;
    int splits = 1, chunk = 0;
    bwd_gather_geometry(V, n, dev.num_cu, &splits, &chunk);

    BwdArgs P{x, m, ga, gp, n, eps2, chunk, nullptr, gx, gm};
    if (splits == 1) {
        if (fault_injected("launch")) return fail(NBODY_ERROR_LAUNCH_FAILED, "injected launch fault");
        prof_mark(stream, 0);
        hipLaunchKernelGGL(V.direct, dim3(iblocks, 1), dim3(V.block), 0, stream, P);
        prof_mark(stream, 1);
        return check_launch(V.name);
    }
    void *ws = nullptr;
    nbody_status st = arena.get(dev, stream, sizeof(float4) * (size_t)splits * n, &ws);
    if (st != NBODY_OK) return st;
    P.partial = static_cast<float4 *>(ws);
    if (fault_injected("launch")) return fail(NBODY_ERROR_LAUNCH_FAILED, "injected launch fault");
    prof_mark(stream, 0);
    hipLaunchKernelGGL(V.partial, dim3(iblocks, splits), dim3(V.block), 0, stream, P);
    prof_mark(stream, 1);
    st = check_launch(V.name);
    if (st != NBODY_OK) return st;
    hipLaunchKernelGGL(backward_reduce_kernel, dim3((n + 255) / 256), dim3(256), 0, stream,
                       P.partial, splits, n, gx, gm);
    return check_launch("backward_reduce");
}

}  // namespace nbody
