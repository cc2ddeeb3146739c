// k_scan64.hip -- the FP64 form of the scan on the FP64 matrix cores.
//
// chi2(d, q) = ||W_q (d - S_q)||^2 (Eq. (1) in factor form, Algorithm 2's
// arithmetic in FP64) for a tile of universes against a chunk of grid points,
// with Algorithm 1's strict-"<" running minimum in grid order.
//
// Contraction.  Per grid point the residual r = d - S_q is formed in FP64
// exactly as Algorithm 2 does (one rounding; r = 0 exactly when d = S_q), and
// y = W_q r is computed on v_mfma_f64_4x4x4f64, whose four 4x4x4 blocks sit at
// lanes 16 k + 4 blk + {row | column}: A[i][k] at lane 16k + 4blk + i, B[k][j]
// at 16k + 4blk + j, D[i][j] at 16i + 4blk + j.  A is one 4 x 4 tile of W_q
// (the same in all four blocks), B holds four bins of 16 universes (four per
// block), D a 4-row block of y for them.  Only the tiles on or below the
// diagonal are issued (N = 57: 105 tiles and a lead column on the vector ALUs,
// 1680 + 57 MACs per evaluation for 1653 algorithmic).  A wave carries two
// sets of 16 universes, so every tile read from LDS feeds two MFMAs; a lane's
// accumulators hold one row of each 4-row block, chi2 is the lane's sum of
// squares plus a butterfly over the four row lanes (lanes l, l ^ 16, l ^ 32,
// l ^ 48), which adds the same operands in the same order in all of them.
//
// Schedule.  On gfx950 a vector instruction takes 4 cycles of a SIMD that the
// FP64 MFMAs (16 cycles each) cannot use, and every change from MFMAs to vector
// work and back 8 more, whatever the instruction.  The point's vector work
// (residuals, lead products, squares, minimum: about 105 instructions at
// N = 57) is therefore gathered into one phase per group of kF64RowGroup row
// blocks, four at N = 57, with nothing but MFMAs and LDS reads between them;
// working group by group keeps one group's accumulators live instead of all
// row blocks' and so leaves the registers (168) for three waves per SIMD, and
// a point's butterfly and minimum wait for the next point's first phase.
// Measured on 100 x 100 points, N = 57, 64 x 2000 universes: 72.2 ms with the
// vector work between the tiles (about 50 changes per point), 67.4 ms so;
// groups of five 68.3, seven 71.4 and all fourteen row blocks 73.1 ms (two
// waves per SIMD for the last two).  Bound: FP64 matrix rate; 3360 of the about
// 3800 cycles a wave spends per point are MFMAs.
//
// Records are double-buffered in LDS (direct global -> LDS loads issued one
// grid point ahead, one barrier per point).  The blocks of one universe tile
// split the grid into chunks; with several chunks each writes its (minimum,
// first q reaching it) to part[chunk][u], the chunk holding p writes
// chi2_p, and k_fp64_merge takes the minimum over the chunks in grid order
// with the same strict "<" -- the sequential scan's result exactly.
#include "fc_internal.h"

namespace fcx {

namespace {

constexpr int kF64Waves = 4;                       // waves per block
constexpr int kF64Sets = 2;                        // sets of 16 universes per wave
constexpr int kF64Univ = 16 * kF64Sets * kF64Waves;  // universes per block (128)
constexpr size_t kF64PartsMax = size_t(2) << 30;      // bytes of chunk partials at most
// Partials past 2 MiB are mapped anew on each call of a caller that waits in
// between: 36 us, about 32 points of a full chip (2000 universes x 400 points of
// 20 bins: 80 chunks 75 us, 64 chunks 41 us).
constexpr int64_t kF64PartsSoft = int64_t(2) << 20;
constexpr double kF64PartsCost = 32.0;

constexpr int kF64Ahead = 2;  // tile pairs read from LDS ahead of their MFMAs

// Sum of x over the lanes l, l ^ 16, l ^ 32, l ^ 48 for two values a (set 0)
// and b (set 1): lanes < 32 get set 0's sum, lanes >= 32 set 1's.  The upper
// half of a is swapped with the lower half of b, then 16-lane rows pair up
// through a swizzle (lane l reads lane l ^ 16), which runs on the LDS unit
// and so takes no vector-ALU time from the FP64 MFMAs.
__device__ __forceinline__ double f64_row_sum(double a, double b)
{
    const uint2 ua = __builtin_bit_cast(uint2, a), ub = __builtin_bit_cast(uint2, b);
    const auto lo = __builtin_amdgcn_permlane32_swap(ua.x, ub.x, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(ua.y, ub.y, false, false);
    const double a2 = __builtin_bit_cast(double, make_uint2(lo[0], hi[0]));
    const double b2 = __builtin_bit_cast(double, make_uint2(lo[1], hi[1]));
    const double h = a2 + b2;  // lane l < 32: a_l + a_{l+32}; lane l >= 32: b_{l-32} + b_l
    const uint2 uh = __builtin_bit_cast(uint2, h);
    // bit-mode swizzle: and 0x1f, or 0, xor 0x10 within each 32-lane half
    const uint32_t sx = (uint32_t)__builtin_amdgcn_ds_swizzle((int)uh.x, 0x401F);
    const uint32_t sy = (uint32_t)__builtin_amdgcn_ds_swizzle((int)uh.y, 0x401F);
    return h + __builtin_bit_cast(double, make_uint2(sx, sy));
}

template <int N>
__global__ __launch_bounds__(64 * kF64Waves) __attribute__((amdgpu_waves_per_eu(3))) void
k_scan_f64m(const uint4 *__restrict__ R64, const double *__restrict__ d,
            const int64_t *__restrict__ p_idx, int64_t K, int64_t q0, int64_t nq,
            int64_t n_utiles, int64_t q_per_chunk, Fp64Part *__restrict__ part,
            double *__restrict__ dchi2, double *__restrict__ chi2_min,
            int64_t *__restrict__ argmin, double *__restrict__ chi2_p)
{
    constexpr int NB = f64_nb(N), P = f64_pad(N), NBE = f64_nbe(N), L = f64_lead(N);
    constexpr int K0 = f64_k0(N), NG = f64_ngroup(N), NPAIR = f64_npair(N);
    constexpr int L1 = L > 0 ? L : 1, S2 = kF64Sets;
    constexpr int REC = f64_rec_units(N);  // 16-byte units per record
    constexpr int LEADU = (f64_lead_double(N) - f64_sig_double(N)) / 2;
    __shared__ uint4 lds[2][REC];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wbase = __builtin_amdgcn_readfirstlane(tid & ~63);
    const int64_t utile = blockIdx.x % n_utiles, chunk = blockIdx.x / n_utiles;
    const int64_t qb = q0 + chunk * q_per_chunk;
    const int64_t qe = (qb + q_per_chunk < q0 + nq) ? qb + q_per_chunk : q0 + nq;
    const int64_t ubase = utile * kF64Univ + (int64_t)wave * 16 * kF64Sets;

    if (qb < qe)
        record_to_lds_sbase<REC, 64 * kF64Waves>(R64 + qb * (int64_t)REC, lds[0], tid, wbase);

    // stage the universes of both sets: bin 4 kb + lane/16 - P of universe
    // lane%16, and the lead bins of the same universe (loads from clamped,
    // in-bounds addresses; padding bins and idle lanes select 0)
    double dv[S2][NB], dl[S2][L1];
#pragma unroll
    for (int c = 0; c < S2; ++c) {
        const int64_t u = ubase + 16 * c + (lane & 15);
        const bool act = u < K;
        const double *du = d + (act ? u : K - 1) * N;
#pragma unroll
        for (int kb = K0; kb < NB; ++kb) {
            const int j = 4 * kb + (lane >> 4) - P;
            const double v = du[j < 0 ? 0 : j];
            dv[c][kb] = (act && j >= 0) ? v : 0.0;
        }
#pragma unroll
        for (int b = 0; b < L; ++b) dl[c][b] = act ? du[b] : 0.0;
    }
    // the universe this lane tracks after the row butterfly; grid points are
    // below 2^31, so a true point outside that range meets none (-2: nor the
    // empty fold before the first point)
    const int64_t u_own = ubase + 16 * (lane >> 5) + (lane & 15);
    const bool own_act = u_own < K;
    const int64_t p = own_act ? p_idx[u_own] : -1;
    const int pi = (p >= 0 && p < (int64_t(1) << 31)) ? (int)p : -2;
    double best = __builtin_inf(), cp = __builtin_nan("");
    int qbest = -1;
    // sums of squares of the previous point, folded in the next point's first
    // vector phase (NaN before the first: it passes no "<")
    double sq[S2];
#pragma unroll
    for (int c = 0; c < S2; ++c) sq[c] = __builtin_nan("");
    const auto fold = [&](int q) {
        const double chi2 = f64_row_sum(sq[0], sq[1]);
        if (__builtin_amdgcn_ballot_w64(q == pi)) cp = (q == pi) ? chi2 : cp;
        if (chi2 < best) {
            best = chi2;
            qbest = q;
        }
    };

    const int tpos = 4 * (lane >> 4) + (lane & 3), spos = (lane >> 4) * (NBE / 2);
    const int qei = (int)qe, qbi = qb < qe ? (int)qb : qei;
    // (restrict: the reads of `cur` need not wait for the loads into `nxt`)
    const auto point = [&](int q, const uint4 *__restrict__ cur, uint4 *__restrict__ nxt) {
        wait_record_loads();
        __syncthreads();  // record q is in cur; every wave is done with nxt
        if (q + 1 < qei)
            record_to_lds_sbase<REC, 64 * kF64Waves>(R64 + (int64_t)(q + 1) * REC, nxt, tid,
                                                     wbase);
        const double2 *tl = reinterpret_cast<const double2 *>(cur) + tpos;
        const double2 *sg = reinterpret_cast<const double2 *>(cur) + f64_sig_double(N) / 2 + spos;
        const double *s_lead = reinterpret_cast<const double *>(cur) + f64_sig_double(N);
        double2 af[NPAIR > 0 ? NPAIR : 1];  // tile pairs
        double2 sv[NBE / 2];                // S_q at the lane's bins
        double2 wl[L1][NBE / 2];            // lead columns at the lane's rows
        double sb[L1], rl[S2][L1];          // S_q and residuals of the lead bins
        double r[S2][NB], acc[S2][NB];
        const auto squares = [&](auto r0, auto r1) {
            static_for<decltype(r0)::value, decltype(r1)::value>([&](auto rc) {
                constexpr int x = decltype(rc)::value;
#pragma unroll
                for (int c = 0; c < S2; ++c)
                    sq[c] = x ? fma(acc[c][x], acc[c][x], sq[c]) : acc[c][x] * acc[c][x];
            });
        };
        // (a bin count with lead columns only, no tiles, still has its one group)
        static_for<0, (NG > 0 ? NG : 1)>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            // rows R0 .. R1-1; bins first needed here: KA .. R1-1; tiles T0 .. T1-1
            constexpr int R0 = g ? f64_group_r0(N, g) : 0;
            constexpr int R1 = NG > 0 ? f64_group_r0(N, g + 1) : NB;
            constexpr int KA = g ? R0 : K0;
            constexpr int T0 = f64_group_t0(N, g), T1 = f64_group_t0(N, g + 1);

            // this phase's LDS reads, ahead of its vector work
            if constexpr (g == 0)
                static_for<0, L>([&](auto bc) {
                    constexpr int b = decltype(bc)::value;
                    sb[b] = s_lead[(P + b) * NBE];  // S_q[b]: bin block 0, lane group P + b
                });
            static_for<0, NBE / 2>([&](auto kc) {
                constexpr int k = decltype(kc)::value, first = 2 * k > K0 ? 2 * k : K0;
                if constexpr (first >= KA && first < R1) sv[k] = sg[k];
                if constexpr ((2 * k >= R0 || (g > 0 && 2 * k + 1 == R0)) && 2 * k < R1)
                    static_for<0, L>([&](auto bc) {
                        constexpr int b = decltype(bc)::value;
                        wl[b][k] = sg[LEADU + b * 2 * NBE + k];
                    });
            });
            static_for<(T0 + 1) / 2, (T0 + 1) / 2 + kF64Ahead>([&](auto xc) {
                constexpr int x = decltype(xc)::value;
                if constexpr (2 * x < T1) af[x] = tl[x * 16];
            });
            __builtin_amdgcn_sched_barrier(0);

            // the vector phase: the last point's minimum or the last group's
            // squares, this group's new residuals, its lead products
            if constexpr (g == 0) {
                fold(q - 1);
                static_for<0, L>([&](auto bc) {
                    constexpr int b = decltype(bc)::value;
#pragma unroll
                    for (int c = 0; c < S2; ++c) rl[c][b] = dl[c][b] - sb[b];
                });
            } else {
                squares(std::integral_constant<int, (g > 1 ? f64_group_r0(N, g - 1) : 0)>{},
                        std::integral_constant<int, R0>{});
            }
            static_for<KA, R1>([&](auto kc) {
                constexpr int kb = decltype(kc)::value;
#pragma unroll
                for (int c = 0; c < S2; ++c)
                    r[c][kb] = dv[c][kb] - ((kb & 1) ? sv[kb / 2].y : sv[kb / 2].x);
            });
            if constexpr (L > 0)
                static_for<R0, R1>([&](auto rc) {
                    constexpr int x = decltype(rc)::value;
                    static_for<0, L>([&](auto bc) {
                        constexpr int b = decltype(bc)::value;
                        const double w = (x & 1) ? wl[b][x / 2].y : wl[b][x / 2].x;
#pragma unroll
                        for (int c = 0; c < S2; ++c)
                            acc[c][x] = b ? fma(w, rl[c][b], acc[c][x]) : w * rl[c][b];
                    });
                });
            __builtin_amdgcn_sched_barrier(0);

            // the group's tiles
            static_for<T0, T1>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                constexpr int kb = f64_tile_kb(N, t), x = f64_tile_r(N, t);
                constexpr int ahead = t / 2 + kF64Ahead;
                if constexpr (t % 2 == 0 && ahead >= (T0 + 1) / 2 + kF64Ahead && 2 * ahead < T1)
                    af[ahead] = tl[ahead * 16];
                const double a = (t & 1) ? af[t / 2].y : af[t / 2].x;
#pragma unroll
                for (int c = 0; c < S2; ++c) {
                    if constexpr (kb == 0)
                        acc[c][x] = __builtin_amdgcn_mfma_f64_4x4x4f64(a, r[c][kb], 0.0, 0, 0, 0);
                    else
                        acc[c][x] =
                            __builtin_amdgcn_mfma_f64_4x4x4f64(a, r[c][kb], acc[c][x], 0, 0, 0);
                }
                if constexpr (t & 1) __builtin_amdgcn_sched_barrier(0);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        squares(std::integral_constant<int, (NG > 1 ? f64_group_r0(N, NG - 1) : 0)>{},
                std::integral_constant<int, NB>{});
    };
    int buf = 0;
    for (int q = qbi; q < qei; ++q, buf ^= 1) point(q, lds[buf], lds[buf ^ 1]);
    if (qbi < qei) fold(qei - 1);
    if (!own_act || (lane & 16)) return;  // one lane per universe writes
    const int64_t q_min = qbest >= 0 ? (int64_t)qbest : p;
    if (part) {
        part[chunk * K + u_own] = Fp64Part{best, q_min};
        if (p >= qb && p < qe) chi2_p[u_own] = cp;
        return;
    }
    if (chi2_min) chi2_min[u_own] = best;
    if (argmin) argmin[u_own] = q_min;
    if (chi2_p) chi2_p[u_own] = cp;
    dchi2[u_own] = cp - best;
}

}  // namespace

// Merge of the FP64 chunks: one wave per universe.  Lane l takes chunks l,
// l + 64, ... in grid order with the strict "<", then the wave reduces the 64
// (value, q) pairs by shuffles, keeping the lower q among equal values: the
// chunks partition the grid in order, so that is the earlier chunk, and the
// result is the sequential scan's.  Chunk values are never NaN (a NaN chi2
// never passes "<"), and a chunk with no finite value reports (+inf, p).  A
// true point outside [0, G) was owned by no chunk: chi2_p = NaN, whatever its
// element holds.  chi2_min and argmin may be nullptr; chi2_p holds the owners'
// values on entry.
__global__ __launch_bounds__(256) void k_fp64_merge(const Fp64Part *__restrict__ part,
                                                   int64_t n_chunks, const int64_t *__restrict__ p_idx,
                                                   int64_t K, int64_t G, double *__restrict__ dchi2,
                                                   double *__restrict__ chi2_min,
                                                   int64_t *__restrict__ argmin,
                                                   double *__restrict__ chi2_p)
{
    const int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (u >= K) return;  // uniform per wave
    const int64_t p = p_idx[u];
    double best = __builtin_inf();
    int64_t qbest = p;
    for (int64_t c = lane; c < n_chunks; c += 64) {
        const Fp64Part x = part[c * K + u];
        if (x.v < best) {
            best = x.v;
            qbest = x.q;
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const double ov = __shfl_xor(best, off, 64);
        const int64_t oq = __shfl_xor(qbest, off, 64);
        if (ov < best || (ov == best && oq < qbest)) {
            best = ov;
            qbest = oq;
        }
    }
    if (lane != 0) return;
    const double cp = (p >= 0 && p < G) ? chi2_p[u] : __builtin_nan("");
    if (chi2_min) chi2_min[u] = best;
    if (argmin) argmin[u] = qbest;
    chi2_p[u] = cp;
    dchi2[u] = cp - best;
}

namespace {

template <int N>
hipError_t launch_f64m_n(const fc_grid *g, int64_t K, const double *d, const int64_t *p_idx,
                          Fp64Part *scratch, size_t scratch_bytes, double *dchi2,
                          double *chi2_min, int64_t *argmin, double *chi2_p, hipStream_t st)
{
    static const int slots =
        resident_slots(reinterpret_cast<const void *>(&k_scan_f64m<N>), 64 * kF64Waves);
    const int64_t G = g->G;
    const int64_t tiles = (K + kF64Univ - 1) / kF64Univ;
    const int64_t chunk_bytes = (int64_t)sizeof(Fp64Part) * K;
    ChunkRule rule = kFp64Chunks;
    rule.soft_chunks = std::max<int64_t>(1, kF64PartsSoft / chunk_bytes);
    rule.soft_cost = kF64PartsCost;
    const ScanGeometry sg =
        scan_geometry(tiles, tiles, G, slots, (int64_t)kF64PartsMax / chunk_bytes, rule);
    int64_t chunks = sg.n_qchunks, qpc = sg.q_per_chunk;
    // the partials must fit the scratch (library-owned or the caller's)
    const int64_t max_chunks = (int64_t)(scratch_bytes / (sizeof(Fp64Part) * (size_t)K));
    Fp64Part *part = nullptr;
    bool own = false;
    if (chunks > 1) {
        if (scratch) {
            if (chunks > max_chunks) {
                chunks = max_chunks < 1 ? 1 : max_chunks;
                qpc = (G + chunks - 1) / chunks;
                chunks = (G + qpc - 1) / qpc;
            }
            if (chunks > 1) part = scratch;
        } else {
            hipError_t e = hipMallocAsync(reinterpret_cast<void **>(&part),
                                          sizeof(Fp64Part) * (size_t)chunks * (size_t)K, st);
            if (e != hipSuccess) return e;
            own = true;
        }
    }
    if (chunks <= 1) {
        chunks = 1;
        qpc = G;
    }
    const int64_t blocks = sg.n_utiles * chunks;
    {
        ProfScope prof(st, "k_scan_f64m");
        hipLaunchKernelGGL(k_scan_f64m<N>, dim3((unsigned)blocks), dim3(64 * kF64Waves), 0, st,
                           g->R64, d, p_idx, K, (int64_t)0, G, sg.n_utiles, qpc, part, dchi2,
                           chi2_min, argmin, chi2_p);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && part) {
        hipLaunchKernelGGL(k_fp64_merge, dim3((unsigned)((K + 3) / 4)), dim3(256), 0, st, part,
                           chunks, p_idx, K, G, dchi2, chi2_min, argmin, chi2_p);
        e = hipGetLastError();
    }
    if (own) {
        const hipError_t ef = hipFreeAsync(part, st);
        if (e == hipSuccess) e = ef;
    }
    return e;
}

}  // namespace

hipError_t launch_scan_fp64(const fc_grid *g, int64_t K, const double *d, const int64_t *p_idx,
                            double *dchi2, double *chi2_min, int64_t *argmin, double *chi2_p,
                            hipStream_t st, Fp64Part *scratch, size_t scratch_bytes)
{
    if (K <= 0) return hipSuccess;
    switch (g->N) {
#define FC_CASE(n)                                                                                \
    case n:                                                                                       \
        return launch_f64m_n<n>(g, K, d, p_idx, scratch, scratch_bytes, dchi2, chi2_min, argmin,  \
                                chi2_p, st);
#define FC_CASE8(b) FC_CASE(b + 1) FC_CASE(b + 2) FC_CASE(b + 3) FC_CASE(b + 4) \
                    FC_CASE(b + 5) FC_CASE(b + 6) FC_CASE(b + 7) FC_CASE(b + 8)
        FC_CASE8(0) FC_CASE8(8) FC_CASE8(16) FC_CASE8(24) FC_CASE8(32) FC_CASE8(40) FC_CASE8(48)
        FC_CASE8(56)
#undef FC_CASE8
#undef FC_CASE
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fcx
