// k_gen.hip -- universes drawn on the device.
//
// Section 2, steps 1-2 of the per-universe procedure: the prediction S(p) at
// the true point is fluctuated into a fake data vector d.  Here d is Poisson
// counts around S(p) plus a correlated Gaussian fractional systematic,
//     d_i = n_i + S_p[i] * (L_F g)_i,   n_i ~ Poisson(S_p[i]),  g ~ N(0, I),
// with L_F the Cholesky factor of the fractional covariance F, so that
// Cov(d) = diag(S_p) + F o (S_p S_p^T), the covariance the scan assumes.
//
// Every random number comes from a counter-based stream, so a universe
// depends only on (seed, p, j) and any batching of the work gives the same
// values:
//   Philox4x64-10 (Salmon, Moraes, Dror and Shaw, SC'11), key (seed, 0);
//   block b of purpose t (0 Poisson, 1 normal) for point p, universe j, bin i
//   has counter (j, p, i << 32 | t << 28 | b, 0);
//   a 64-bit word w is the uniform ((w >> 11) + 0.5) 2^-53 in (0, 1).
// Poisson(lambda): 0 for lambda = 0; the multiplication method below 10 (the
// product of successive uniforms, first at or below exp(-lambda), at most
// 1024 of them); Hormann's transformed rejection with squeeze (PTRS, 1993)
// from 10 up (attempt t uses words 2(t%2), 2(t%2)+1 of block t/2, at most 512
// attempts, then floor(lambda)).  Normal: Box-Muller, sqrt(-2 ln u0)
// cos(2 pi u1) from words 0 and 1 of the bin's normal block.  A mean that is
// negative, NaN or infinite gives count -1 and d = NaN.
//
// A block takes a tile of up to kGenRows universes, one thread per (universe, bin).
// Most Poisson draws end at the first attempt's squeeze; with a lane per bin of
// one universe, some lane of every wave needed the exact test (two logarithms
// and lgamma) and the whole wave waited through it up to four times.  The draws
// that the squeeze does not settle therefore go to a list in LDS and are drawn
// afterwards with full waves; a tile with at most one draw a thread has nothing
// to gain from that and draws at once.  The constants of the squeeze depend on
// (p, bin) alone and are tabulated for a tile's first point where segments are
// long; L_F sits in LDS by columns (consecutive bins, consecutive addresses).
// Bound: FP64 and 64-bit integer vector arithmetic (two Philox blocks of 20
// 64 x 64 products each).  16 x 10 000 universes, N = 57: 1.12 ms with one wave per
// universe, 0.47 ms so.  Short segments, one universe each of 400 / 4000 / 40 000
// points, N = 57, stream of calls: 16.8 / 37.5 / 319 us with one wave per
// universe, 19.5 / 43.7 / 203 through a table of the tile's first point alone,
// 14.2 / 32.9 / 171 so.
//
// The arithmetic is FP64 without contraction, in the order written, so the
// counts are the same integers on any IEEE machine that evaluates
// exp/log/lgamma to within an ulp (a decision flips only if a uniform lands
// within rounding of a boundary).
#include "fc_internal.h"

#include <algorithm>

namespace fcx {

#pragma clang fp contract(off)

__device__ __forceinline__ void philox4x64_10(uint64_t x[4], uint64_t k0, uint64_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t m0 = 0xD2E7470EE14C6C93ull, m1 = 0xCA5A826395121157ull;
        const uint64_t hi0 = __umul64hi(m0, x[0]), lo0 = m0 * x[0];
        const uint64_t hi1 = __umul64hi(m1, x[2]), lo1 = m1 * x[2];
        const uint64_t y0 = hi1 ^ x[1] ^ k0, y2 = hi0 ^ x[3] ^ k1;
        x[0] = y0;
        x[1] = lo1;
        x[2] = y2;
        x[3] = lo0;
        k0 += 0x9E3779B97F4A7C15ull;
        k1 += 0xBB67AE8584CAA73Bull;
    }
}

__device__ __forceinline__ void stream_block(uint64_t seed, int64_t p, int64_t j, int i,
                                             uint32_t purpose, uint32_t b, uint64_t w[4])
{
    w[0] = (uint64_t)j;
    w[1] = (uint64_t)p;
    w[2] = ((uint64_t)(uint32_t)i << 32) | ((uint64_t)purpose << 28) | (uint64_t)b;
    w[3] = 0;
    philox4x64_10(w, seed, 0);
}

__device__ __forceinline__ double unit_open(uint64_t w)
{
    return ((double)(w >> 11) + 0.5) * 0x1.0p-53;
}

// PTRS constants of a mean (functions of sqrt(lambda) only)
struct Ptrs {
    double A, B, vr;
};
__device__ __forceinline__ Ptrs ptrs_constants(double lam)
{
    Ptrs c;
    c.B = 0.931 + 2.53 * sqrt(lam);
    c.A = -0.059 + 0.02483 * c.B;
    c.vr = 0.9277 - 3.6224 / (c.B - 2.0);
    return c;
}
// PTRS candidate of the words (wu, wv): its count kf, with us and V
__device__ __forceinline__ double ptrs_candidate(const Ptrs &c, double lam, uint64_t wu,
                                                 uint64_t wv, double &us, double &V)
{
    const double U = unit_open(wu) - 0.5;
    V = unit_open(wv);
    us = 0.5 - fabs(U);
    return floor((2.0 * c.A / us + c.B) * U + lam + 0.43);
}
__device__ __forceinline__ bool ptrs_squeeze(const Ptrs &c, double us, double V)
{
    return us >= 0.07 && V <= c.vr;
}

// Poisson count for bin i of universe j at point p (-1: no valid mean).
__device__ __forceinline__ int64_t poisson_draw(double lam, uint64_t seed, int64_t p, int64_t j, int i)
{
    if (!(lam >= 0.0) || __builtin_isinf(lam)) return -1;
    if (lam == 0.0) return 0;
    uint64_t w[4];
    if (lam < 10.0) {
        const double floor_p = exp(-lam);
        double prod = 1.0;
        int64_t k = 0;
        for (uint32_t b = 0; b < 256; ++b) {
            stream_block(seed, p, j, i, 0, b, w);
            for (int e = 0; e < 4; ++e) {
                prod = prod * unit_open(w[e]);
                if (prod <= floor_p) return k;
                k = k + 1;
            }
        }
        return k;
    }
    const Ptrs c = ptrs_constants(lam);
    const double ll = log(lam);
    const double ia = 1.1239 + 1.1328 / (c.B - 3.4);
    for (uint32_t t = 0; t < 512; ++t) {
        if ((t & 1u) == 0u) stream_block(seed, p, j, i, 0, t >> 1, w);
        const int h = 2 * (int)(t & 1u);
        double us, V;
        const double kf = ptrs_candidate(c, lam, w[h], w[h + 1], us, V);
        if (ptrs_squeeze(c, us, V)) return (int64_t)kf;        // accept
        if (kf < 0.0 || (us < 0.013 && V > us)) continue;      // outside the hat
        const double lhs = log(V * ia / (c.A / (us * us) + c.B));
        const double rhs = -lam + kf * ll - lgamma(kf + 1.0);
        if (lhs <= rhs) return (int64_t)kf;
    }
    return (int64_t)floor(lam);
}

__device__ __forceinline__ double normal_draw(uint64_t seed, int64_t p, int64_t j, int i)
{
    uint64_t w[4];
    stream_block(seed, p, j, i, 1, 0, w);
    const double u0 = unit_open(w[0]), u1 = unit_open(w[1]);
    return sqrt(-2.0 * log(u0)) * cos(6.283185307179586 * u1);
}

// Cholesky factor of the fractional covariance, one 64-lane block, lane i
// owning row i (right-looking, in LDS).  flag = 1 if positive definite.
__global__ __launch_bounds__(64) void k_chol_frac(const double *__restrict__ F, int N,
                                                  double *__restrict__ LF, int *__restrict__ flag)
{
    __shared__ double A[kMaxBins * kMaxBins];
    const int i = threadIdx.x;
    for (int e = i; e < N * N; e += 64) A[e] = F[e];
    __syncthreads();
    bool ok = true;
    for (int c = 0; c < N; ++c) {
        const double piv = A[c * N + c];
        if (!(piv > 0.0)) {  // every lane read the same pivot
            ok = false;
            break;
        }
        const double lcc = sqrt(piv);
        __syncthreads();
        if (i == c) A[c * N + c] = lcc;
        if (i > c && i < N) A[i * N + c] = A[i * N + c] / lcc;
        __syncthreads();
        if (i > c && i < N) {
            const double lic = A[i * N + c];
            for (int k = c + 1; k <= i; ++k) A[i * N + k] = A[i * N + k] - lic * A[k * N + c];
        }
        __syncthreads();
    }
    if (i < N)
        for (int k = 0; k < N; ++k) LF[i * N + k] = (ok && k <= i) ? A[i * N + k] : 0.0;
    if (i == 0) *flag = ok ? 1 : 0;
}

// Largest k in [0, n) with seg_off[k] <= r (seg_off non-decreasing).
__device__ __forceinline__ int64_t segment_of(const int64_t *__restrict__ seg_off, int64_t n,
                                              int64_t r)
{
    int64_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (seg_off[mid] <= r)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

constexpr int kGenRows = 16;  // universes of a block at most

// How a tile's Poisson draws go: all at once (at most a draw a thread), or the
// squeeze first and the list then, with the constants of the tile's first point
// from a table (draws of another point go to the list) or each draw's own.
enum GenMode { kGenAtOnce, kGenTable, kGenOwn };

// One tile of at most kGenRows universes a block (a loop over tiles lets the
// compiler keep the library functions' constants in registers across it: 555
// us at three waves per SIMD with spills, against 466).
template <GenMode MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_gen_universes(
    const double *__restrict__ S64, const double *__restrict__ LF, int N, int64_t G,
    int64_t n_pts, const int64_t *__restrict__ p, const int64_t *__restrict__ seg_off,
    const int64_t *__restrict__ u_first, uint64_t seed, int64_t row0, int64_t K, int tile_rows,
    double *__restrict__ d, int64_t *__restrict__ p_idx, int32_t *__restrict__ counts)
{
    __shared__ double lft[kMaxBins * kMaxBins];  // L_F by columns: lft[l N + i]
    __shared__ double gs[kGenRows][kMaxBins];    // normals
    __shared__ int64_t ns[kGenRows][kMaxBins];   // counts
    __shared__ Ptrs cs[kMaxBins];                // squeeze constants of point p_cs
    __shared__ double lam_s[kMaxBins];           // its means
    __shared__ int64_t pk_s[kGenRows], j_s[kGenRows];
    __shared__ uint16_t slow[kGenRows * kMaxBins];  // draws the squeeze left open
    __shared__ int n_slow;
    const int tid = threadIdx.x;
    const int64_t r0 = row0 + (int64_t)blockIdx.x * tile_rows;
    if (r0 >= K) return;
    const int rows = (int)(K - r0 < tile_rows ? K - r0 : tile_rows);
    // L_F by all threads, or where a call is few tiles and its time a tile's, by
    // three waves while the first looks up the rows
    constexpr int kLook = MODE == kGenAtOnce ? 64 : 0;
    if (tid >= kLook)
        for (int e = tid - kLook; e < N * N; e += 256 - kLook) lft[(e % N) * N + e / N] = LF[e];
    if (tid < rows) {
        const int64_t k = segment_of(seg_off, n_pts, r0 + tid);
        const int64_t pk = p[k];
        pk_s[tid] = (pk >= 0 && pk < G) ? pk : -1;
        j_s[tid] = (u_first ? u_first[k] : 0) + (r0 + tid - seg_off[k]);
        if (p_idx) p_idx[r0 + tid] = pk_s[tid];
    }
    if (tid == 0) n_slow = 0;
    __syncthreads();
    const int64_t p_cs = MODE == kGenTable ? pk_s[0] : -2;  // the tabulated point
    if constexpr (MODE == kGenTable) {
        if (tid < N && p_cs >= 0) {
            lam_s[tid] = S64[p_cs * N + tid];
            cs[tid] = ptrs_constants(lam_s[tid]);
        }
        __syncthreads();
    }
    // normals, and the counts that the first attempt's squeeze settles
    for (int e = tid; e < rows * N; e += 256) {
        const int u = e / N, i = e - u * N;
        const int64_t pk = pk_s[u], j = j_s[u];
        double g = 0.0;
        int64_t n = -1;
        if (pk >= 0) {
            g = normal_draw(seed, pk, j, i);
            bool open = true;
            if (MODE == kGenOwn || (MODE == kGenTable && pk == p_cs)) {
                const double lam = MODE == kGenTable ? lam_s[i] : S64[pk * N + i];
                if (lam >= 10.0 && !__builtin_isinf(lam)) {
                    const Ptrs c = MODE == kGenTable ? cs[i] : ptrs_constants(lam);
                    uint64_t w[4];
                    stream_block(seed, pk, j, i, 0, 0, w);
                    double us, V;
                    const double kf = ptrs_candidate(c, lam, w[0], w[1], us, V);
                    if (ptrs_squeeze(c, us, V)) {
                        n = (int64_t)kf;
                        open = false;
                    }
                }
            }
            if (MODE != kGenAtOnce && open)
                slow[atomicAdd(&n_slow, 1)] = (uint16_t)(u * kMaxBins + i);
        }
        gs[u][i] = g;
        ns[u][i] = n;
    }
    __syncthreads();
    if constexpr (MODE == kGenAtOnce) {
        if (tid < rows * N) {
            const int u = tid / N, i = tid - u * N;
            if (pk_s[u] >= 0)
                ns[u][i] = poisson_draw(S64[pk_s[u] * N + i], seed, pk_s[u], j_s[u], i);
        }
    } else {
        for (int e = tid; e < n_slow; e += 256) {
            const int u = slow[e] / kMaxBins, i = slow[e] % kMaxBins;
            ns[u][i] = poisson_draw(S64[pk_s[u] * N + i], seed, pk_s[u], j_s[u], i);
        }
    }
    __syncthreads();
    // z_i = sum_{l <= i} L_F[i][l] g_l, increasing l
    for (int e = tid; e < rows * N; e += 256) {
        const int u = e / N, i = e - u * N;
        double z = 0.0;
#pragma unroll 8
        for (int l = 0; l < N; ++l) z = z + lft[l * N + i] * gs[u][l];  // L_F is 0 past i
        const int64_t pk = pk_s[u], n = ns[u][i];
        const double lam = pk < 0 ? 0.0 : (pk == p_cs ? lam_s[i] : S64[pk * N + i]);
        d[(r0 + u) * N + i] = (n < 0) ? __builtin_nan("") : (double)n + lam * z;
        if (counts) counts[(r0 + u) * N + i] = (int32_t)n;
    }
}

hipError_t launch_chol_frac(const double *F, int N, double *LF, int *flag, hipStream_t st)
{
    hipLaunchKernelGGL(k_chol_frac, dim3(1), dim3(64), 0, st, F, N, LF, flag);
    return hipGetLastError();
}

hipError_t launch_gen_universes(const fc_grid *g, int64_t n_pts, const int64_t *p,
                                const int64_t *seg_off, const int64_t *u_first, uint64_t seed,
                                int64_t K, double *d, int64_t *p_idx, int32_t *counts,
                                hipStream_t st)
{
    // (Times of a call in a stream of calls, N = 57.)  As small tiles as one round of
    // resident blocks takes (4000 universes, one a point: tiles of 5 in 1.04 rounds
    // 41 us, of 6 in 0.87 32 us); few universes a tile a CU, of at most four rows
    // (tiles of 1 / 2 / 4 rows: 1000 of one point 17.9 / 13.0 / 11.1 us, 400 of as
    // many points 14.3 / 15.8 / 17.3).
    static const int slots =  // queried once (thread-safe)
        resident_slots(reinterpret_cast<const void *>(&k_gen_universes<kGenTable>), 256);
    const int64_t few = std::min<int64_t>(4, std::max<int64_t>(1, (K + 64) / 256));
    const int rows = (int)std::min<int64_t>(kGenRows, std::max(few, (K + slots - 1) / slots));
    // The list pays where there are more draws than threads (1000 of one point,
    // tiles of four rows: 12.9 us through it, 11.1 at once); the table where
    // most tiles have one point, judged by the mean segment, as their lengths are
    // known on the device only (table against own constants: 16 segments of
    // 10 000 480 / 488 us, 300 of 250 246 / 247, 400 of 100 145 / 141).
    const auto kernel = rows * g->N <= 256             ? k_gen_universes<kGenAtOnce>
                        : K / n_pts >= 16 * kGenRows ? k_gen_universes<kGenTable>
                                                     : k_gen_universes<kGenOwn>;
    const int64_t per_launch = (int64_t(1) << 22) * rows;  // blocks x 256 inside 32 bits
    for (int64_t row0 = 0; row0 < K; row0 += per_launch) {
        const int64_t n = K - row0 < per_launch ? K - row0 : per_launch;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((n + rows - 1) / rows)), dim3(256), 0, st,
                           g->S64, g->LF64, g->N, g->G, n_pts, p, seg_off, u_first, seed, row0, K,
                           rows, d, p_idx, counts);
    }
    return hipGetLastError();
}

}  // namespace fcx
