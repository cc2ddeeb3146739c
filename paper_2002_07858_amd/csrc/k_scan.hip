// k_scan.hip -- the chi^2 grid scan (Eq. (1) inside Algorithm 1's loops).
//
// FP32 form (the hot kernel).  Eq. (1) is evaluated in factor form,
//     chi2(d, q) = ||W_q (d - S_q)||^2,   W_q = L_q^{-1} (lower triangular),
// which equals (d-S_q)^T Sigma_q^{-1} (d-S_q).  For a fixed q and a tile of
// universes this is a dense contraction Z = W_q R (R = bins x universes),
// done on the matrix cores with v_mfma_f32_4x4x1_16b_f32: one universe per
// lane, one bin per instruction, the 4-row slice of W_q broadcast to all 16
// lane blocks.  The 4-row granularity covers the lower triangle with little
// waste (N = 57: 1740 issued multiply-adds per evaluation for 1653 needed),
// and each lane ends with its own universe's rows, so chi2 is a lane-local
// sum of squares followed by a strict-"<" running minimum.  On this chip a
// vector instruction takes 4 cycles of a SIMD that the FP32 MFMAs (8 cycles
// each) cannot use and every change from MFMAs to vector work and back 8 more,
// and one wave alone issues an MFMA every 11.5 cycles, two every 8.5, three
// every 8.3.  The rows are therefore contracted in groups of kFp32RowGroup row
// blocks: one vector phase per group, and one group's accumulators live
// instead of all, which leaves the offset form below 128 registers (four waves
// per SIMD, two before) and the residual form's residuals formed once per
// point at two waves per SIMD.  The launch is then bound by power: the matrix
// cores are 92 % busy at 2.22 GHz (85 % at 2.31 GHz before; offset form, 100 x
// 100 points, N = 57, 256 x 2000 universes: 142.1 -> 137.3 ms; residual form,
// 27 000 points x 20 000 universes: 17.4 -> 16.9 ms; three waves per SIMD with
// the universes' low parts in LDS 16.9-17.1 ms).
//
// Work decomposition: a 256-thread block owns 256 universes (one per lane)
// and walks a contiguous range of grid points in list order.  Each lane
// keeps its universe's residual sources in registers; the block
// double-buffers one record per grid point in LDS (W_q slices, S_q and the
// correction C_q), bringing the next record in with direct global -> LDS
// loads while the waves contract the current one, with one barrier per grid
// point.  Ranges of the same universes are merged with a
// 64-bit atomicMin on keys (FP32 chi2 bits above q), which reproduces
// Algorithm 1's rule that the lowest q wins exact ties whatever the split.
#include "fc_internal.h"

#include <algorithm>
#include <utility>

namespace fcx {

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float pick(const float4 &v, int c)
{
    return c == 0 ? v.x : (c == 1 ? v.y : (c == 2 ? v.z : v.w));
}

// A universe as its lane carries it through its range of grid points.  It
// is held as d = dh + dl: dh = float(d) and dl, the rest, as FP16
// scaled by a per-universe power of two 2^e (so that the largest |dl| 2^e
// lies in [2^14, 2^15)); dl 2^e keeps 11 bits, so d is carried to 35 bits,
// and the residual costs one subtraction and one mixed FP16/FP32 FMA.
template <int N>
struct Fp32Lane {
    float dh[N];
    uint32_t dl[(N + 1) / 2];  // dl 2^e as FP16, bins 2i (low half) and 2i+1 (high half)
    float dl_scale;            // 2^-e
};

// r = dl 2^-e + t with dl taken from one FP16 half of a packed register: the
// compiler folds the half selection and the conversion into one
// mixed-precision FMA (v_fma_mix_f32).
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
template <int HI>
__device__ __forceinline__ float fma_mix_dl(uint32_t dl2, float scale, float t)
{
    const half2_t h = __builtin_bit_cast(half2_t, dl2);
    return __builtin_fmaf((float)h[HI], scale, t);
}

// Sums of squares over row blocks B0 .. B1-1 into the lane's four FP32 chains
// (one per row of a block; the P padding rows of block 0 are zero and skipped).
// A single block's are added up as FMAs.
template <int P, int B0, int B1, int NS>
__device__ __forceinline__ void fp32_squares(const v4f (&acc)[NS], float (&part)[4])
{
    if constexpr (NS == 1) {
        const v4f z = acc[0];
        part[1] = part[3] = 0.0f;
        part[0] = P < 1 ? fmaf(z[0], z[0], z[1] * z[1]) : 0.0f;
        part[2] = P < 3 ? fmaf(z[2], z[2], z[3] * z[3]) : z[3] * z[3];
        if constexpr (P == 1) part[2] = fmaf(z[1], z[1], part[2]);
        return;
    }
    static_for<B0, B1>([&](auto bc) {
        constexpr int b = decltype(bc)::value;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (b == 0)
                part[j] = (j >= P) ? acc[0][j] * acc[0][j] : 0.0f;
            else
                part[j] = fmaf(acc[b][j], acc[b][j], part[j]);
        }
    });
}

// The squares of z = W_q r + c0 of one grid point, group by group: part's four
// chains add up to chi2.  wl: the record's A slices at this lane, c0: the rows'
// starts (the same in every lane), both in LDS; r: the lane's universe at
// every bin.  Padded bins left of the shift (k' < P) are zero and generate no
// code.
template <int N>
__device__ __forceinline__ void fp32_contract(const float4 *wl, const float4 *c0,
                                              const float (&r)[N], float (&part)[4])
{
    constexpr int NS = n_ksteps(N), P = fp32_pad(NS, N), NG = fp32_ngroup(NS);
    constexpr int NA = n_groups_from_ns(NS);
    float4 a[NA];  // four A registers each, read 32 pairs ahead
    v4f acc[NS];
    a[0] = wl[0];
    static_for<0, NG>([&](auto gc) {
        constexpr int g = decltype(gc)::value;
        constexpr int B0 = fp32_group_b0(NS, g), B1 = fp32_group_b0(NS, g + 1);
        static_for<B0, B1>([&](auto bc) {
            constexpr int b = decltype(bc)::value;
            const float4 cv = c0[b];
            acc[b] = v4f{cv.x, cv.y, cv.z, cv.w};
        });
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (g > 0) {  // while the starts arrive
            fp32_squares<P, fp32_group_b0(NS, g - 1), B0>(acc, part);
            __builtin_amdgcn_sched_barrier(0);
        }
        static_for<fp32_group_i0(NS, g), fp32_group_i0(NS, g + 1)>([&](auto ic) {
            constexpr int i = decltype(ic)::value, t = fp32_pair_at(NS, i), v = i / 16;
            constexpr int kp = fp32_pair_kp(NS, t), b = fp32_pair_b(NS, t);
            if constexpr (i % 64 == 32 && i / 64 + 1 < NA) a[i / 64 + 1] = wl[(i / 64 + 1) * 64];
            if constexpr (kp >= P)
                acc[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(pick(a[i / 64], v % 4), r[kp - P],
                                                            acc[b], 4, i % 16, 0);
            // keeps the scheduler from hoisting later operands (registers)
            if constexpr (i % 16 == 15) __builtin_amdgcn_sched_barrier(0);
        });
        __builtin_amdgcn_sched_barrier(0);
    });
    fp32_squares<P, fp32_group_b0(NS, NG - 1), NS>(acc, part);
}

// The lane's running minimum over the grid points of its range, and chi2 at
// its true point.  A point's chains are folded after the next point's copies
// have been issued; the NaN start passes no "<" and meets no true point.
struct Fp32Min {
    float part[4];
    float best, cp;
    uint32_t qbest;
    int p;  // the universe's true point (-2: none that a grid point can meet)

    __device__ __forceinline__ explicit Fp32Min(int64_t p_own)
    {
        part[0] = part[1] = part[2] = part[3] = cp = __builtin_nanf("");
        best = __builtin_inff();
        qbest = 0xffffffffu;
        p = (p_own >= 0 && p_own < (int64_t(1) << 31)) ? (int)p_own : -2;
    }
    __device__ __forceinline__ void fold(int q)
    {
        const float chi2 = (part[0] + part[1]) + (part[2] + part[3]);
        if (__builtin_amdgcn_ballot_w64(q == p)) cp = (q == p) ? chi2 : cp;
        if (chi2 < best) {
            best = chi2;
            qbest = (uint32_t)q;
        }
    }
    // merge universe u's range [qb, qe) into its state
    __device__ __forceinline__ void merge(int64_t u, int64_t qb, int64_t qe,
                                          unsigned long long *keys, double *chi2_p) const
    {
        if (p >= qb && p < qe) chi2_p[u] = (double)cp;
        if (best < __builtin_inff())
            atomicMin(&keys[u], ((unsigned long long)__float_as_uint(best) << 32) |
                                    (unsigned long long)qbest);
    }
};

// One work item (a tile of 256 universes x a range of grid points) in the
// residual form: d - S_q is formed per bin and grid point.
template <int N>
__device__ __forceinline__ void fp32_item(const ScanItem &it,
                                          uint4 (&lds)[2][rec_units(n_ksteps(N))])
{
    constexpr int NS = n_ksteps(N), NWU = rec_w_units(NS);
    constexpr int REC = rec_units(NS);  // A groups + 512 B of S and C
    constexpr int THREADS = 64 * kWavesPerBlock;

    const uint4 *__restrict__ R32 = it.R;
    const double *__restrict__ d = it.d;
    const int64_t K = it.K;
    const int tid = threadIdx.x;
    const int64_t u = it.u0 + tid;  // this lane's universe
    const int64_t qb = it.qb, qe = it.qe;
    if (qb >= qe) return;  // uniform per block

    Fp32Lane<N> L;
    // residual sources d = dh + dl 2^-e (zero past K; lanes past K still take
    // part in the copies and barriers).  The rest d - dh is exact in FP64.
    float rest[N];
    float big = 0.0f;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double v = (u < K) ? d[u * N + k] : 0.0;
        L.dh[k] = (float)v;
        rest[k] = (float)(v - (double)L.dh[k]);
        big = fmaxf(big, fabsf(rest[k]));
    }
    // largest |rest| 2^e in [2^14, 2^15); e clamped so that 2^-e stays a
    // normal FP32 number (rests that small are below FP16's reach and vanish)
    int e = (big > 0.0f) ? 14 - ilogbf(big) : 0;
    e = e < -100 ? -100 : (e > 100 ? 100 : e);
    L.dl_scale = ldexpf(1.0f, -e);
#pragma unroll
    for (int i = 0; i < (N + 1) / 2; ++i) {
        const _Float16 lo = (_Float16)ldexpf(rest[2 * i], e);
        const _Float16 hi = (2 * i + 1 < N) ? (_Float16)ldexpf(rest[2 * i + 1], e) : (_Float16)0.0f;
        L.dl[i] = (uint32_t)__builtin_bit_cast(uint16_t, lo) |
                  ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
    }
    Fp32Min m((u < K) ? (it.p_idx ? it.p_idx[u] : it.p) : -1);

    const int lane = tid & 63, wbase = __builtin_amdgcn_readfirstlane(tid & ~63);
    record_to_lds_sbase<REC, THREADS>(R32 + qb * REC, lds[0], tid, wbase);
    const int qei = (int)qe;
    // (restrict: the reads of `cur` need not wait for the loads into `nxt`)
    const auto point = [&](int q, const uint4 *__restrict__ cur, uint4 *__restrict__ nxt) {
        // the packed FP16 parts are re-presented to the compiler at every grid
        // point, so that their FP32 conversions stay inside the mixed FMAs
        // instead of being hoisted out of the grid loop into extra registers
#pragma unroll
        for (int i = 0; i < (N + 1) / 2; ++i) asm volatile("" : "+v"(L.dl[i]));
        wait_record_loads();
        __syncthreads();  // record q is in cur; every wave is done with nxt
        if (q + 1 < qei)
            record_to_lds_sbase<REC, THREADS>(R32 + (int64_t)(q + 1) * REC, nxt, tid, wbase);
        __builtin_amdgcn_sched_barrier(0);
        m.fold(q - 1);
        // the residuals of every bin in one phase, the signal's FP32 part from
        // LDS (uniform reads, kAhead of four bins ahead; through the scalar
        // cache they would make the LDS reads wait for the scalar loads)
        constexpr int kAhead = 4;
        const float4 *sg = reinterpret_cast<const float4 *>(cur + NWU);
        float r[N];
        float4 s[NS];
        static_for<0, (kAhead < NS ? kAhead : NS)>([&](auto xc) {
            constexpr int x = decltype(xc)::value;
            s[x] = sg[x];
        });
        static_for<0, NS>([&](auto xc) {
            constexpr int x = decltype(xc)::value;
            if constexpr (x + kAhead < NS) s[x + kAhead] = sg[x + kAhead];
            static_for<4 * x, (4 * x + 4 < N ? 4 * x + 4 : N)>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                r[k] = fma_mix_dl<k & 1>(L.dl[k / 2], L.dl_scale, L.dh[k] - pick(s[x], k % 4));
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        // accumulators start at C_q (the same four rows in every lane)
        fp32_contract<N>(reinterpret_cast<const float4 *>(cur) + lane,
                         reinterpret_cast<const float4 *>(cur + NWU) + 16, r, m.part);
    };
    int buf = 0;
    for (int q = (int)qb; q < qei; ++q, buf ^= 1) point(q, lds[buf], lds[buf ^ 1]);
    m.fold(qei - 1);
    if (u < K) m.merge(u, qb, qe, it.keys, it.chi2_p);
}

template <int N>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_scan_fp32(
    const uint4 *__restrict__ R32, const double *__restrict__ d,
    const int64_t *__restrict__ p_idx, int64_t K, int64_t q_lo, int64_t q_hi, int64_t n_utiles,
    int64_t q_per_chunk, unsigned long long *__restrict__ keys, double *__restrict__ chi2_p)
{
    __shared__ uint4 lds[2][rec_units(n_ksteps(N))];
    ScanItem it;
    it.R = R32;
    it.d = d;
    it.p_idx = p_idx;
    it.p = -1;
    it.keys = keys;
    it.chi2_p = chi2_p;
    it.off = nullptr;
    it.K = K;
    it.N = N;
    it.ed = 0;
    const int64_t utile = blockIdx.x % n_utiles;
    const int64_t qchunk = blockIdx.x / n_utiles;
    it.u0 = utile * (int64_t)kFp32UnivPerBlock;
    it.qb = q_lo + qchunk * q_per_chunk;
    it.qe = (it.qb + q_per_chunk < q_hi) ? it.qb + q_per_chunk : q_hi;
    fp32_item<N>(it, lds);
}

// Serving: a persistent-style launch over a table of items (any mix of
// requests and grids with this bin count).  Resident blocks take items in
// turn from an atomic counter until the table is exhausted; the table is
// finite and fixed at launch, so every block reaches the exit.
template <int N>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_serve_fp32(
    const ScanItem *__restrict__ items, int n_items, int *__restrict__ counter)
{
    __shared__ uint4 lds[2][rec_units(n_ksteps(N))];
    __shared__ int cur;
    for (;;) {
        if (threadIdx.x == 0) cur = atomicAdd(counter, 1);
        __syncthreads();
        const int i = cur;
        __syncthreads();
        if (i >= n_items) break;
        fp32_item<N>(items[i], lds);
        __syncthreads();
    }
}

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

__global__ __launch_bounds__(256) void k_init_keys(int64_t K, unsigned long long *__restrict__ keys,
                                                  double *__restrict__ chi2_p, double chi2_p_fill)
{
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= K) return;
    keys[u] = kKeyNone;
    chi2_p[u] = chi2_p_fill;
}

// Decode the keys.  chi2_min may be the key buffer itself (decoded in place:
// each thread reads its key before it writes the same element); chi2_min and
// argmin may be nullptr.  A universe
// with no finite chi2 keeps Algorithm 1's initial state and gets a NaN dchi2,
// and so does one whose true point is outside [0, p_limit) when p_limit > 0.
__global__ __launch_bounds__(256) void k_finalize(int64_t K, const int64_t *__restrict__ p_idx,
                                                 int64_t p_uniform, int64_t p_limit,
                                                 const unsigned long long *keys, double *chi2_min,
                                                 int64_t *__restrict__ argmin,
                                                 const double *__restrict__ chi2_p,
                                                 double *__restrict__ dchi2)
{
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= K) return;
    const unsigned long long key = keys[u];
    const uint32_t hi = (uint32_t)(key >> 32);
    double cmin, dc;
    int64_t am;
    if (hi >= 0x7f800000u) {  // no chi2 < +inf was seen: Algorithm 1's initial state
        cmin = __builtin_inf();
        am = p_idx ? p_idx[u] : p_uniform;
        dc = __builtin_nan("");
    } else {
        cmin = (double)__uint_as_float(hi);
        am = (int64_t)(uint32_t)(key & 0xffffffffu);
        dc = chi2_p[u] - cmin;
        if (p_limit > 0) {
            const int64_t pu = p_idx ? p_idx[u] : p_uniform;
            if (pu < 0 || pu >= p_limit) dc = __builtin_nan("");
        }
    }
    if (chi2_min) chi2_min[u] = cmin;
    if (argmin) argmin[u] = am;
    dchi2[u] = dc;
}

// ---------------------------------------------------------------------------
// Resident block slots of a kernel on the current device: CUs x blocks per CU
// from the occupancy calculator.
int resident_slots(const void *kernel, int block_threads)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
        return 512;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block_threads, 0) !=
            hipSuccess ||
        per_cu <= 0)
        per_cu = 2;
    return cus * per_cu;
}

// Grid chunks of a scan.  All blocks of a launch take about the same time, one
// chunk each, so the launch takes rounds(c) = ceil(tiles c / slots) of them and
// a half-empty last round is lost; c is the count that minimises
//     rounds(c) (points per chunk + kChunkCost),
// kChunkCost being a block's start (staging its universes) in points.  Chunks
// are at most kChunkMax points long, so that the blocks that share a chunk stay
// close and the L2 serves the later readers of each record, and at least
// kChunkMin, which sets how far a small scan spreads over the CUs.  (FP64, 1000
// tiles x 10 000 points on 768 slots: 5 chunks in 6.5 rounds 67.6 ms, 23 in
// 29.95 rounds 65.2 ms; split FP16, 20 tiles x 216 000 points on 512 slots: 106
// chunks in 4.1 rounds 12.7 ms, 128 in 5.0 rounds 11.0 ms.)
ScanGeometry scan_geometry(int64_t n_utiles, int64_t tiles, int64_t G, int slots,
                           int64_t max_chunks)
{
    constexpr int64_t kChunkMax = 2048, kChunkMin = 4, kChunkCost = 2;
    ScanGeometry sg;
    sg.n_utiles = n_utiles;
    // blocks x 256 work-items stay well inside the 32-bit dispatch size
    const int64_t fit = (int64_t(1) << 23) / std::max<int64_t>(n_utiles, 1);
    const int64_t cap = std::max<int64_t>(1, std::min(max_chunks, fit));
    const int64_t lo = std::min(cap, (G + kChunkMax - 1) / kChunkMax);
    const int64_t hi = std::min(cap, std::max(lo, std::min(G / kChunkMin, 2 * lo + 512)));
    int64_t best = INT64_MAX;
    for (int64_t c = lo; c <= hi; ++c) {
        const int64_t q = (G + c - 1) / c, n = (G + q - 1) / q;
        const int64_t cost = (tiles * n + slots - 1) / slots * (q + kChunkCost);
        if (cost < best) {
            best = cost;
            sg.q_per_chunk = q;
            sg.n_qchunks = n;
        }
    }
    return sg;
}

template <int N>
static hipError_t launch_fp32_n(const fc_grid *g, int64_t K, const double *d, const int64_t *p_idx,
                                int64_t q0, int64_t nq, unsigned long long *keys, double *chi2_p,
                                hipStream_t st)
{
    // resident block slots: queried once per instantiation (thread-safe)
    static const int slots =
        resident_slots(reinterpret_cast<const void *>(&k_scan_fp32<N>), 64 * kWavesPerBlock);
    const int64_t tiles = (K + kFp32UnivPerBlock - 1) / kFp32UnivPerBlock;
    const ScanGeometry sg = scan_geometry(tiles, tiles, nq, slots, nq);
    const int64_t blocks = sg.n_utiles * sg.n_qchunks;
    ProfScope prof(st, "k_scan_fp32");
    hipLaunchKernelGGL((k_scan_fp32<N>), dim3((unsigned)blocks), dim3(64 * kWavesPerBlock), 0, st,
                       g->R32, d, p_idx, K, q0, q0 + nq, sg.n_utiles, sg.q_per_chunk, keys, chi2_p);
    return hipGetLastError();
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
    const ScanGeometry sg = scan_geometry(n_tiles, tiles, nq, slots, nq);
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

template <int N>
static hipError_t launch_serve_fp32_n(const ScanItem *items, int n_items, int *counter, int blocks,
                                      hipStream_t st)
{
    hipLaunchKernelGGL((k_serve_fp32<N>), dim3((unsigned)blocks), dim3(256), 0, st, items, n_items,
                       counter);
    return hipGetLastError();
}

template <int N>
static int serve_slots_fp32_n()
{
    // resident block slots: queried once per instantiation (thread-safe)
    static const int slots =
        resident_slots(reinterpret_cast<const void *>(&k_serve_fp32<N>), 256);
    return slots;
}

int serve_fp32_univ_per_item() { return kFp32UnivPerBlock; }

// One instantiation per bin count: the padding shift and the skipped pairs
// are compile-time constants of the kernel.
#define FC_EACH_N(X)                                                                            \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)       \
    X(17) X(18) X(19) X(20) X(21) X(22) X(23) X(24) X(25) X(26) X(27) X(28) X(29) X(30) X(31) \
    X(32) X(33) X(34) X(35) X(36) X(37) X(38) X(39) X(40) X(41) X(42) X(43) X(44) X(45) X(46) \
    X(47) X(48) X(49) X(50) X(51) X(52) X(53) X(54) X(55) X(56) X(57) X(58) X(59) X(60) X(61) \
    X(62) X(63) X(64)

hipError_t launch_serve_fp32(int N, const ScanItem *items, int n_items, int *counter, int blocks,
                             hipStream_t st)
{
    switch (N) {
#define FC_CASE(n) \
    case n: return launch_serve_fp32_n<n>(items, n_items, counter, blocks, st);
        FC_EACH_N(FC_CASE)
#undef FC_CASE
    default: return hipErrorInvalidValue;
    }
}

int serve_slots_fp32(int N)
{
    switch (N) {
#define FC_CASE(n) \
    case n: return serve_slots_fp32_n<n>();
        FC_EACH_N(FC_CASE)
#undef FC_CASE
    default: return 512;
    }
}

hipError_t launch_scan_fp32(const fc_grid *g, int64_t K, const double *d, const int64_t *p_idx,
                            int64_t q0, int64_t nq, unsigned long long *keys, double *chi2_p,
                            hipStream_t st)
{
    switch (g->N) {
#define FC_CASE(n) \
    case n: return launch_fp32_n<n>(g, K, d, p_idx, q0, nq, keys, chi2_p, st);
        FC_EACH_N(FC_CASE)
#undef FC_CASE
    default: return hipErrorInvalidValue;
    }
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
#undef FC_EACH_N

hipError_t launch_init_keys(int64_t K, unsigned long long *keys, double *chi2_p, hipStream_t st,
                            double chi2_p_fill)
{
    const int64_t blocks = (K + 255) / 256;
    hipLaunchKernelGGL(k_init_keys, dim3((unsigned)blocks), dim3(256), 0, st, K, keys, chi2_p,
                       chi2_p_fill);
    return hipGetLastError();
}

hipError_t launch_finalize(int64_t K, const int64_t *p_idx, const unsigned long long *keys,
                           double *chi2_min, int64_t *argmin, const double *chi2_p, double *dchi2,
                           hipStream_t st, int64_t p_uniform, int64_t p_limit)
{
    const int64_t blocks = (K + 255) / 256;
    hipLaunchKernelGGL(k_finalize, dim3((unsigned)blocks), dim3(256), 0, st, K, p_idx, p_uniform,
                       p_limit, keys, chi2_min, argmin, chi2_p, dchi2);
    return hipGetLastError();
}

}  // namespace fcx
