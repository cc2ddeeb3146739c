// k_scan_fp32.h -- the FP32 form of the chi^2 grid scan (Eq. (1) inside Algorithm
// 1's loops): the contraction and one work item, shared by k_scan.hip (scan),
// k_scan_pts.hip (scan of universes grouped by true point) and k_serve.hip
// (request serving), which are compiled in parallel.
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
// 27 000 points x 20 000 universes: 17.4 -> 16.9 ms, 216 000 points the same at
// 128.6 ms; three waves per SIMD with the universes' low parts in LDS
// 16.9-17.1 ms).
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
#pragma once
#include "fc_internal.h"

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

// One instantiation per bin count: the padding shift and the skipped pairs
// are compile-time constants of the kernel.
#define FC_EACH_N(X)                                                                            \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)       \
    X(17) X(18) X(19) X(20) X(21) X(22) X(23) X(24) X(25) X(26) X(27) X(28) X(29) X(30) X(31) \
    X(32) X(33) X(34) X(35) X(36) X(37) X(38) X(39) X(40) X(41) X(42) X(43) X(44) X(45) X(46) \
    X(47) X(48) X(49) X(50) X(51) X(52) X(53) X(54) X(55) X(56) X(57) X(58) X(59) X(60) X(61) \
    X(62) X(63) X(64)

}  // namespace fcx
