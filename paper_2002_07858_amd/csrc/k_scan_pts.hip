// k_scan_pts.hip -- the FP32 scan of universes grouped by true point
// (k_scan_fp32.h), its offset table and its tiles.
#include "k_scan_fp32.h"

#include <algorithm>

namespace fcx {

// Scan of universes grouped by true point, in the offset form: with
// e = d - S_p rounded to FP32 once,
//     W_q (d - S_q) = W_q e + T_pq,    T_pq = W_q (S_p - S_q),
// and T_pq (FP64 arithmetic on the FP32 factor, rounded once) is the
// accumulators' start, read from a table built before the scan.  The MFMAs
// take e straight from registers, so the grid loop has no vector work besides
// the squares and the minimum.  Tiles of
// B = kPtsTile universes never straddle segments: segment s owns the dense
// tile ids [tile_start[s], tile_start[s+1]), tile_start[s+1] - tile_start[s] =
// ceil(len_s / B) (a prefix sum built before the launch), all below
// floor(K / B) + n_pts.  Each block scans one tile (its waves share the true
// point, so one offset-table row per grid point serves them all) over a range
// of grid points.  Blocks are dispatched round-robin over the 8 XCDs (block b
// runs on XCD b mod 8), so block b = xcd + 8 (m + 8 (j + J c)) is given tile
// 8 (xcd + 8 j) + m of grid chunk c: eight consecutive tiles (a segment's,
// mostly) run on one XCD at the same time and share its L2 for the offset
// rows and the records, and the XCDs get equal shares of the tiles.
// The grid points scanned are [q_lo, q_hi): the whole grid, or one slice of it
// when the grid is split over several launches or devices.  Segments whose
// true point is outside the grid do nothing.
template <int N>
__global__ __launch_bounds__(kPtsTile) __attribute__((amdgpu_waves_per_eu(3))) void k_scan_fp32_pts(
    const uint4 *__restrict__ R32, const double *__restrict__ S64, const double *__restrict__ d,
    int64_t G, int64_t n_pts, const int64_t *__restrict__ p, const int64_t *__restrict__ seg_off,
    const int64_t *__restrict__ tile_start, const float *__restrict__ T, int64_t groups_per_xcd,
    int64_t q_lo, int64_t q_hi, int64_t q_per_chunk, int64_t K,
    unsigned long long *__restrict__ keys, double *__restrict__ chi2_p)
{
    constexpr int NS = n_ksteps(N);
    constexpr int REC = rec_units(NS);
    constexpr int NR = 4 * NS;
    constexpr int THREADS = kPtsTile;
    __shared__ uint4 lds[2][REC], tb[2][16];
    const int64_t b = blockIdx.x;
    const int64_t xcd = b % 8, k = b / 8;
    const int64_t member = k % 8, rest = k / 8;
    const int64_t group = xcd + 8 * (rest % groups_per_xcd);
    const int64_t tile = 8 * group + member;
    const int64_t qb = q_lo + (rest / groups_per_xcd) * q_per_chunk;
    const int64_t qe = (qb + q_per_chunk < q_hi) ? qb + q_per_chunk : q_hi;
    if (tile >= tile_start[n_pts]) return;  // uniform per block
    // the tile's segment: the largest s with tile_start[s] <= tile (uniform)
    int64_t lo = 0, hi = n_pts - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (tile_start[mid] <= tile)
            lo = mid;
        else
            hi = mid - 1;
    }
    const int64_t seg = lo;
    const int64_t i = tile - tile_start[seg];
    const int64_t s0 = seg_off[seg], s1 = seg_off[seg + 1];
    const int64_t pp = p[seg];
    if (qb >= qe || pp < 0 || pp >= G) return;  // uniform per block
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wbase = __builtin_amdgcn_readfirstlane(tid & ~63);
    const int64_t u = s0 + kPtsTile * i + tid;
    // (the row must also lie in [0, K): offsets that break their contract
    // read and write nothing outside the arrays)
    const bool act = u < s1 && u >= 0 && u < K;

    // offset rows of this segment, one of 4 ns floats per grid point of
    // [q_lo, q_hi); the block's first wave copies them beside the records
    const float *__restrict__ trow = T + (seg * (q_hi - q_lo) + (qb - q_lo)) * NR;
    record_to_lds_sbase<REC, THREADS>(R32 + qb * REC, lds[0], tid, wbase);
    if (wbase == 0)
        record_to_lds_sbase<NS, 64>(reinterpret_cast<const uint4 *>(trow), tb[0], lane, 0);
    const double *__restrict__ sp = S64 + pp * N;  // uniform: scalar loads
    float e[N];
    static_for<0, N>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        e[k] = act ? (float)(d[u * N + k] - sp[k]) : 0.0f;
        if constexpr (k % 16 == 15) __builtin_amdgcn_sched_barrier(0);  // 16 loads in flight
    });
    Fp32Min m(act ? pp : -1);
    const int qei = (int)qe;
    // (restrict: the reads of `cur` and `tcur` need not wait for the loads
    // into the other buffers)
    const auto point = [&](int q, const uint4 *__restrict__ cur, uint4 *__restrict__ nxt,
                           const uint4 *__restrict__ tcur, uint4 *__restrict__ tnxt) {
        wait_record_loads();
        __syncthreads();  // record q is in cur; every wave is done with nxt
        trow += NR;
        if (q + 1 < qei) {
            record_to_lds_sbase<REC, THREADS>(R32 + (int64_t)(q + 1) * REC, nxt, tid, wbase);
            if (wbase == 0)
                record_to_lds_sbase<NS, 64>(reinterpret_cast<const uint4 *>(trow), tnxt, lane, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        m.fold(q - 1);
        fp32_contract<N>(reinterpret_cast<const float4 *>(cur) + lane,
                         reinterpret_cast<const float4 *>(tcur), e, m.part);
    };
    int buf = 0;
    for (int q = (int)qb; q < qei; ++q, buf ^= 1)
        point(q, lds[buf], lds[buf ^ 1], tb[buf], tb[buf ^ 1]);
    m.fold(qei - 1);
    if (act) m.merge(u, qb, qe, keys, chi2_p);
}

// Dense tile ids of the points scan: tile_start[0] = 0, tile_start[s+1] =
// tile_start[s] + ceil((seg_off[s+1] - seg_off[s]) / kPtsTile).  One block;
// segments in chunks of 1024 with a running carry.
__global__ __launch_bounds__(1024) void k_tile_prefix(int64_t n_pts,
                                                      const int64_t *__restrict__ seg_off,
                                                      int64_t *__restrict__ tile_start)
{
    __shared__ int64_t part[1024];
    const int tid = threadIdx.x;
    int64_t carry = 0;
    if (tid == 0) tile_start[0] = 0;
    for (int64_t base = 0; base < n_pts; base += 1024) {
        const int64_t s = base + tid;
        int64_t v = 0;
        if (s < n_pts) {
            const int64_t len = seg_off[s + 1] - seg_off[s];
            v = len > 0 ? (len + kPtsTile - 1) / kPtsTile : 0;
        }
        part[tid] = v;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {  // inclusive scan (Hillis-Steele)
            const int64_t add = tid >= off ? part[tid - off] : 0;
            __syncthreads();
            part[tid] += add;
            __syncthreads();
        }
        if (s < n_pts) tile_start[s + 1] = carry + part[tid];
        carry += part[1023];
        __syncthreads();
    }
}

template <int N>
static hipError_t launch_fp32_pts_n(const fc_grid *g, int64_t n_pts, const int64_t *p,
                                    const int64_t *seg_off, int64_t K, const double *d, int64_t q0,
                                    int64_t nq, const float *T, int64_t *tile_start,
                                    unsigned long long *keys, double *chi2_p, hipStream_t st)
{
    // resident block slots: queried once per instantiation (thread-safe)
    static const int slots =
        resident_slots(reinterpret_cast<const void *>(&k_scan_fp32_pts<N>), kPtsTile);
    const int64_t max_tiles = K / kPtsTile + n_pts;  // bound on the dense tile count
    const int64_t groups_per_xcd = (max_tiles + 63) / 64;
    const int64_t n_tiles = 64 * groups_per_xcd;    // blocks per grid chunk
    // tiles with work if the segments are about equally long (their lengths are
    // known on the device only)
    const int64_t len = (K + n_pts - 1) / n_pts;
    const int64_t tiles = std::min(max_tiles, n_pts * ((len + kPtsTile - 1) / kPtsTile));
    const ScanGeometry sg = scan_geometry(n_tiles, pts_busy_tiles(tiles), nq, slots, nq, kPointsChunks);
    const int64_t blocks = n_tiles * sg.n_qchunks;
    hipLaunchKernelGGL(k_tile_prefix, dim3(1), dim3(1024), 0, st, n_pts, seg_off, tile_start);
    ProfScope prof(st, "k_scan_fp32_pts");
    hipLaunchKernelGGL((k_scan_fp32_pts<N>), dim3((unsigned)blocks), dim3(kPtsTile), 0,
                       st, g->R32, g->S64, d, g->G, n_pts, p, seg_off, tile_start, T, groups_per_xcd,
                       q0, q0 + nq, sg.q_per_chunk, K, keys, chi2_p);
    return hipGetLastError();
}

// Offset table of the FP32 offset form: T[pt][q - q_lo][r'] = sum_k' W'_q[r'][k']
// (S_p - S_q)[k' - P] for the true point p = p[pt] of every segment and every
// grid point q of [q_lo, q_lo + nq), in FP64
// arithmetic on the FP32 factor as the scan uses it (padded rows r' < 4 ns),
// rounded once to FP32; rows of an out-of-range p are zero (such segments take
// the residual form).  One block per grid point (grid-stride): the record's A
// slices are expanded into the transposed dense factor W'^T in LDS (zero above
// the diagonal), and each thread accumulates one 4-row block of one segment,
// bin by bin, from float4 columns of W'^T.
template <int N>
__global__ __launch_bounds__(256) void k_offset_table(const uint4 *__restrict__ R32,
                                                      const double *__restrict__ S64, int64_t G,
                                                      int64_t q_lo, int64_t nq, int64_t n_pts,
                                                      const int64_t *__restrict__ p,
                                                      float *__restrict__ T)
{
    constexpr int NS = n_ksteps(N), P = fp32_pad(NS, N), NR = 4 * NS;
    constexpr int REC = rec_units(NS), NP = fp32_npairs(NS), NG = n_groups_from_ns(NS);
    __shared__ float4 Wt[NR * NS];  // Wt[k'][b] = W'[4b .. 4b+3][k']
    __shared__ double Sq[NR];
    __shared__ unsigned char pk[NP], pb[NP];
    const int tid = threadIdx.x;
    if (tid == 0) {
        int t = 0;  // position in the record
        for (int g = 0; g < fp32_ngroup(NS); ++g) {
            const int b0 = fp32_group_b0(NS, g), b1 = fp32_group_b0(NS, g + 1);
            for (int kp = 0; kp < 4 * b1; ++kp)
                for (int b = max(kp / 4, b0); b < b1; ++b, ++t) {
                    pk[t] = (unsigned char)kp;
                    pb[t] = (unsigned char)b;
                }
        }
    }
    __syncthreads();
    float *wt = reinterpret_cast<float *>(Wt);
    for (int64_t j = blockIdx.x; j < nq; j += gridDim.x) {
        const int64_t q = q_lo + j;
        for (int i = tid; i < NR * NR; i += blockDim.x) wt[i] = 0.0f;
        for (int i = tid; i < NR; i += blockDim.x) Sq[i] = (i >= P) ? S64[q * N + (i - P)] : 0.0;
        __syncthreads();
        const float *rec = reinterpret_cast<const float *>(R32 + q * REC);
        // float f of the A part: register v = 4 (f / 256) + f % 4, lane (f / 4) % 64
        for (int f = tid; f < NG * 256; f += blockDim.x) {
            const int v = 4 * (f / 256) + (f & 3), ln = (f >> 2) & 63;
            const int t = 16 * v + (ln >> 2);
            if (t < NP) wt[pk[t] * NR + 4 * pb[t] + (ln & 3)] = rec[f];
        }
        __syncthreads();
        // one thread per (segment, 4-row block): few segments still use the
        // whole block, and a row's sum runs over k' in ascending order
        for (int64_t w = tid; w < n_pts * NS; w += blockDim.x) {
            const int64_t pt = w / NS;
            const int b = (int)(w - pt * NS);
            const int64_t pp = p[pt];
            double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
            if (pp >= 0 && pp < G) {
                const double *sp = S64 + pp * N - P;
                for (int kp = P; kp < NR; ++kp) {
                    const double dk = sp[kp] - Sq[kp];
                    const float4 wv = Wt[kp * NS + b];
                    a0 = fma((double)wv.x, dk, a0);
                    a1 = fma((double)wv.y, dk, a1);
                    a2 = fma((double)wv.z, dk, a2);
                    a3 = fma((double)wv.w, dk, a3);
                }
            }
            reinterpret_cast<float4 *>(T + (pt * nq + j) * NR)[b] =
                make_float4((float)a0, (float)a1, (float)a2, (float)a3);
        }
        __syncthreads();
    }
}

// Segment expansion: universe u of segment s = max{k : seg_off[k] <= u} gets
// p_idx[u] = p[s].
__global__ __launch_bounds__(256) void k_expand_segments(int64_t K, int64_t n_pts,
                                                         const int64_t *__restrict__ seg_off,
                                                         const int64_t *__restrict__ p,
                                                         int64_t *__restrict__ p_idx)
{
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < K;
         u += (int64_t)gridDim.x * blockDim.x) {
        int64_t lo = 0, hi = n_pts - 1;
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (seg_off[mid] <= u)
                lo = mid;
            else
                hi = mid - 1;
        }
        p_idx[u] = p[lo];
    }
}

template <int N>
static hipError_t launch_offset_table_n(const fc_grid *g, int64_t n_pts, const int64_t *p,
                                        int64_t q0, int64_t nq, float *T, hipStream_t st)
{
    const int64_t blocks = nq < 65536 ? nq : 65536;
    ProfScope prof(st, "k_offset_table");
    hipLaunchKernelGGL((k_offset_table<N>), dim3((unsigned)blocks), dim3(256), 0, st, g->R32, g->S64,
                       g->G, q0, nq, n_pts, p, T);
    return hipGetLastError();
}

hipError_t launch_scan_fp32_points(const fc_grid *g, int64_t n_pts, const int64_t *p,
                                   const int64_t *seg_off, int64_t K, const double *d, int64_t q0,
                                   int64_t nq, const float *T, int64_t *tile_start,
                                   unsigned long long *keys, double *chi2_p, hipStream_t st)
{
    switch (g->N) {
#define FC_CASE(n)                                                                             \
    case n:                                                                                    \
        return launch_fp32_pts_n<n>(g, n_pts, p, seg_off, K, d, q0, nq, T, tile_start, keys, \
                                    chi2_p, st);
        FC_EACH_N(FC_CASE)
#undef FC_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_offset_table(const fc_grid *g, int64_t n_pts, const int64_t *p, int64_t q0,
                               int64_t nq, float *T, hipStream_t st)
{
    switch (g->N) {
#define FC_CASE(n) \
    case n: return launch_offset_table_n<n>(g, n_pts, p, q0, nq, T, st);
        FC_EACH_N(FC_CASE)
#undef FC_CASE
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_expand_segments(int64_t K, int64_t n_pts, const int64_t *seg_off,
                                  const int64_t *p, int64_t *p_idx, hipStream_t st)
{
    int64_t blocks = (K + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_expand_segments, dim3((unsigned)blocks), dim3(256), 0, st, K, n_pts, seg_off,
                       p, p_idx);
    return hipGetLastError();
}

}  // namespace fcx
