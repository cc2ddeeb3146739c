// k_cov_impl.h -- per-grid-point covariance, FP64 Cholesky and inverse factor
// (the kernel template; instantiated per padded bin count NP in the
// k_cov_np_*.hip files, launched from k_cov.hip).
//
// For grid point q (Section 1: M in Eq. (1) is the inverse of a covariance
// carrying statistical and systematic uncertainties):
//     Sigma_q = diag(stat_q) + F o (S_q S_q^T)
//     L_q L_q^T = Sigma_q          right-looking Cholesky, FP64
//     W_q = L_q^{-1}               forward substitution, FP64
// so that Sigma_q^{-1} = W_q^T W_q and chi2 = ||W_q r||^2.  This is the step
// whose conditioning needs FP64; the scan forms only ever see W_q.
//
// One wave per grid point, the matrices in registers as 16 x 16 tiles in the
// layout of v_mfma_f64_16x16x4_f64's output (lane l, register r: row l/16 + 4 r,
// column l%16), bins padded to tiles with the identity's rows and columns.
// Right-looking in panels of four columns, A the trailing part of Sigma_q and S
// the right-hand sides of L W = 1, both lower-triangular in tiles:
//   * the panel's four columns of A go through LDS to a lane per row; column j
//     gives the pivot p = A[j][j], 1/sqrt(p) (the hardware estimate and two
//     Newton steps) and 1/p as its square, m_i = A[i][j] / p, and updates the
//     columns after it in the panel, A[i][k] -= m_i A[k][j];
//   * the tiles right of the panel take all four columns in one MFMA each,
//     A[i][k] += sum_j (-m_ij) A[k][j], j ascending;
//   * the panel's four rows of S go through LDS to a lane per column:
//     w_j = s_j / L[j][j] are rows of W, and the rows below take
//     S[r][i] += sum_j A[r][j] (-w_ji / L[j][j]) in one MFMA per tile.
// The FP64 MFMA adds its four products one after the other, each rounded as an
// FMA, so every element goes through the operations of the column-by-column
// algorithm in their order.  135 MFMAs a point at N = 57; no column of L is
// kept.  W_q's rows go into LDS as they come, packed, and from there to HBM and,
// gathered through a per-N map (fc_internal.h), into each requested record form,
// in 16-byte stores.
//
// Measured at N = 57, 216 000 points: FP64 and FP32 forms (7.8 GB written, 1.6 ms
// at the rate of a large copy) 6.87 ms with a lane per row and one column at a
// time (every column read back through LDS as broadcasts, the LDS 60 % and the
// vector units 47 % busy), 3.63 ms so; split FP16 form 7.40 and 4.15 ms.  The
// bytes do not bound it (a third of them, FP32 records alone, takes 4 % less
// time), nor the matrix cores (23 % busy): of the waves' time 39 % is waiting to
// issue and 25 % for LDS or memory, at the two waves a SIMD that the matrix tiles'
// registers allow, with vector instructions on 35 % of the cycles; the pivots'
// reciprocal roots (57, each after the last panel's update) are one serial chain.
#pragma once
#include <stdint.h>

#include "fc_internal.h"

namespace fcx {

typedef double v4d __attribute__((ext_vector_type(4)));

// LDS doubles of one point: W_q's packed rows, S_q, then two panel buffers of
// four rows of 64 (at the end S_q - fl32(S_q) and S_q - o).
__host__ __device__ constexpr int cov_region(int NP) { return (NP * (NP + 1) / 2 + 1) & ~1; }
constexpr int kCovPanel = 4 * 64;
__host__ __device__ constexpr int cov_lds_doubles(int NP)
{
    return cov_region(NP) + 64 + 2 * kCovPanel;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// hi + lo split of eight FP32 values into two 16-byte fragments (round to
// nearest even for both halves).
template <bool FP16>
__device__ inline void split8(const float (&x)[8], uint4 &hi, uint4 &lo)
{
    if constexpr (FP16) {
        f16x8 h, l;
        for (int e = 0; e < 8; ++e) {
            h[e] = (_Float16)x[e];
            l[e] = (_Float16)(x[e] - (float)h[e]);
        }
        hi = __builtin_bit_cast(uint4, h);
        lo = __builtin_bit_cast(uint4, l);
    } else {
        bf16x8 h, l;
        for (int e = 0; e < 8; ++e) {
            h[e] = (__bf16)x[e];
            l[e] = (__bf16)(x[e] - (float)h[e]);
        }
        hi = __builtin_bit_cast(uint4, h);
        lo = __builtin_bit_cast(uint4, l);
    }
}

// The wave's LDS writes before this are seen by its reads after it (the LDS
// serves a wave in order; this keeps the compiler's order).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double lane_value(double x, int lane)  // lane: uniform
{
    const uint2 u = __builtin_bit_cast(uint2, x);
    return __builtin_bit_cast(double, make_uint2(__builtin_amdgcn_readlane(u.x, lane),
                                                 __builtin_amdgcn_readlane(u.y, lane)));
}

// Map entries of a record's 16-byte units, E elements each: unit lane + 64 b in
// en[b], all read before the record's stores (a load waits for every store
// issued before it).
template <int E>
struct __attribute__((packed, aligned(4))) CovEntries {
    int16_t m[E];
};
template <int E, int B>
__device__ __forceinline__ void cov_entries(const int16_t *__restrict__ map, int units, int lane,
                                            CovEntries<E> (&en)[B])
{
    const CovEntries<E> *me = reinterpret_cast<const CovEntries<E> *>(map);
#pragma unroll
    for (int b = 0; b < B; ++b) en[b] = me[lane + 64 * b < units ? lane + 64 * b : units - 1];
}

// The units themselves: element e comes through its entry from W_q's packed
// rows at Lc or from S_q, `sig` doubles behind them.
template <int E, int B, class Pack>
__device__ __forceinline__ void cov_records(const CovEntries<E> (&en)[B], int units,
                                            const double *Lc, int sig, int lane,
                                            uint4 *__restrict__ rec, Pack pack)
{
#pragma unroll
    for (int b = 0; b < B; ++b) {
        double v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int m = en[b].m[e];
            const double x = Lc[m < 0 ? 0 : (m >= kMapSig ? sig + m - kMapSig : m)];
            v[e] = m < 0 ? 0.0 : x;
        }
        if (lane + 64 * b < units) rec[lane + 64 * b] = pack(v);
    }
}

// One split-form record (see fc_internal.h) from W_q's packed rows in LDS;
// wmax = max |W_q| (FP16 range).  Each fragment element is one gathered W_q
// entry, scaled, rounded to the 16-bit type (hi) or, marked kMapLo, the rest
// of that rounding (lo).
template <bool FP16, int B>
__device__ __forceinline__ void write_split_record(const double *Wl, const double *sdo,
                                                   const CovEntries<8> (&en)[B], int N, int ed,
                                                   double wmax, uint4 *rq, int i)
{
    const int code = split_code(N);
    const int eq = (FP16 && wmax > 0.0) ? 13 - ilogb(wmax) : 0;
    const int nf = code_nfrag(code);
    static_for<0, B>([&](auto fc) {
        constexpr int f = decltype(fc)::value;
        if (f >= nf) return;  // uniform
        float x[8];
        bool lo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int m = en[f].m[e];
            lo[e] = m >= 0 && (m & kMapLo) != 0;
            x[e] = (m < 0) ? 0.0f : (float)ldexp(Wl[m & (kMapLo - 1)], eq);
        }
        uint4 hi, lw;
        split8<FP16>(x, hi, lw);
        const uint32_t *ph = reinterpret_cast<const uint32_t *>(&hi);
        const uint32_t *pl = reinterpret_cast<const uint32_t *>(&lw);
        uint32_t w[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t m0 = lo[2 * h] ? 0x0000ffffu : 0u;
            const uint32_t m1 = lo[2 * h + 1] ? 0xffff0000u : 0u;
            w[h] = (ph[h] & ~(m0 | m1)) | (pl[h] & (m0 | m1));
        }
        rq[f * 64 + i] = make_uint4(w[0], w[1], w[2], w[3]);
    });
    // u_q = W_q (S_q - o) in FP64, in the accumulator's row order [l/16][g][j]
    {
        const int gl = i >> 4, g = (i >> 2) & 3, j = i & 3;
        const int row = split_row0(N, g) + 4 * gl + j;
        double u = 0.0;
        if (g < split_nb(N) && row < split_row0(N, g + 1)) {
            const double *wr = Wl + row * (row + 1) / 2;
#pragma unroll 8
            for (int k = 0; k <= row; ++k) u += wr[k] * sdo[k];
        }
        reinterpret_cast<float *>(rq + code_u_unit(code))[i] = (float)ldexp(-u, eq + ed);
    }
    const int su = code_scale_unit(code), ru = code_rec_units(code);
    if (i == 0) rq[su] = make_uint4(__float_as_uint(ldexpf(1.0f, -2 * (eq + ed))), 0u, 0u, 0u);
    for (int u = su + 1 + i; u < ru; u += 64) rq[u] = make_uint4(0u, 0u, 0u, 0u);
}

// Most 16-byte units a lane holds of each record form, over the bin counts
// N = NP-3 .. NP.
__host__ __device__ constexpr int cov_max4(int a, int b, int c, int d)
{
    const int e = a > b ? a : b, f = c > d ? c : d;
    return e > f ? e : f;
}
__host__ __device__ constexpr int cov_units64(int NP)
{
    return ceil_div(cov_max4(f64_rec_units(NP - 3), f64_rec_units(NP - 2), f64_rec_units(NP - 1),
                             f64_rec_units(NP)),
                    64);
}
__host__ __device__ constexpr int cov_units32(int NP) { return n_groups_from_ns(NP / 4); }
__host__ __device__ constexpr int cov_units16(int NP)
{
    return cov_max4(code_nfrag(split_code(NP - 3)), code_nfrag(split_code(NP - 2)),
                    code_nfrag(split_code(NP - 1)), code_nfrag(split_code(NP)));
}

template <int NP>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) void k_cov_build(
    const double *__restrict__ S64, const double *__restrict__ F, const double *__restrict__ stat,
    const double *__restrict__ off, int N_arg, int64_t G, int stat_mode, uint32_t forms, int ns,
    int ed16, const int16_t *__restrict__ maps, double *__restrict__ W64, uint4 *__restrict__ R64,
    uint4 *__restrict__ R32, uint4 *__restrict__ RB16, uint4 *__restrict__ RH16,
    unsigned long long *__restrict__ bad_q)
{
    static_assert(NP % 4 == 0 && NP >= 4 && NP <= 64, "NP: a multiple of four up to 64");
    constexpr int T = (NP + 15) / 16;  // tiles a side
    extern __shared__ double smem[];
    double *const Lc = smem;                 // W_q's packed rows
    double *const Sl = Lc + cov_region(NP);  // S_q
    double *const P0 = Sl + 64;              // panel buffers [4][64]
    double *const P1 = P0 + kCovPanel;
    const double stat_i =
        ((int)threadIdx.x < N_arg && stat_mode != FC_STAT_PEARSON) ? stat[threadIdx.x] : 0.0;
    const double off_i = ((int)threadIdx.x < N_arg) ? off[threadIdx.x] : 0.0;

    const auto fetch_F = [&](v4d (&A)[T][T], int N, int g, int c) {
        static_for<0, T>([&](auto Kc) {
            constexpr int K = decltype(Kc)::value;
            const int k = 16 * K + c < N ? 16 * K + c : N - 1;
            static_for<K, T>([&](auto Ic) {
                constexpr int I = decltype(Ic)::value;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = 16 * I + g + 4 * r;
                    A[I][K][r] = F[k * N + (row < N ? row : N - 1)];  // F is symmetric
                }
            });
        });
    };
    double s_next = ((int)threadIdx.x < N_arg && (int64_t)blockIdx.x < G)
                        ? S64[(int64_t)blockIdx.x * N_arg + threadIdx.x]
                        : 0.0;
    for (int64_t q = blockIdx.x; q < G; q += gridDim.x) {
        // the lane index and N re-read per point: everything derived from them
        // (addresses and predicates of NP rows) would otherwise be hoisted out
        // of the loop and held in registers across it
        int i = threadIdx.x, N = N_arg;
        asm volatile("" : "+v"(i), "+s"(N));
        const int g = i >> 4, c = i & 15;
        const int16_t *map64 = maps;
        const int16_t *map32 = map64 + 2 * f64_rec_units(N);
        const int16_t *map16 = map32 + 4 * rec_w_units(ns);
        const double si = s_next;
        v4d A[T][T];
        fetch_F(A, N, g, c);
        Sl[i] = si;
        P0[i] = (i < N) ? ((stat_mode == FC_STAT_PEARSON) ? si : stat_i) : 1.0;  // diagonal term
        wave_lds_sync();

        // ---- Sigma_q: tiles (I, K), I >= K ---------------------------------
        v4d S[T][T];
        static_for<0, T>([&](auto Kc) {
            constexpr int K = decltype(Kc)::value;
            const int k = 16 * K + c;
            const double sk = Sl[k], dk = P0[k];
            static_for<K, T>([&](auto Ic) {
                constexpr int I = decltype(Ic)::value;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
#pragma clang fp contract(off)
                    const int row = 16 * I + g + 4 * r;
                    double v = A[I][K][r] * (Sl[row] * sk);  // rounded before the diagonal's sum
                    if (I == T - 1 && (row >= N || k >= N)) v = 0.0;  // (N > NP - 4)
                    if (I == K && row == k) v = v + dk;
                    A[I][K][r] = v;
                }
            });
        });

        // ---- panels of four columns ------------------------------------------
        int bad = 0;  // a pivot <= 0 or NaN (uniform)
        static_for<0, NP / 4>([&](auto pc) {
            constexpr int p = decltype(pc)::value, J = p / 4, pp = p % 4;
            // tile column J of S starts as the identity's
            if constexpr (pp == 0)
                static_for<J, T>([&](auto Rc) {
                    constexpr int R = decltype(Rc)::value;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        S[R][J][r] = (R == J && g + 4 * r == c) ? 1.0 : 0.0;
                });
            // its columns of A, a lane per row (rows above tile J are not used),
            // and its rows of S, a lane per column
            wave_lds_sync();
            if ((c >> 2) == pp)
                static_for<J, T>([&](auto Ic) {
                    constexpr int I = decltype(Ic)::value;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        P0[(c & 3) * 64 + 16 * I + g + 4 * r] = A[I][J][r];
                });
            static_for<0, J + 1>([&](auto Ic) {
                constexpr int I = decltype(Ic)::value;
                P1[g * 64 + 16 * I + c] = S[J][I][pp];
            });
            wave_lds_sync();
            double x[4], w[4], s[4], inv[4], nm[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                x[a] = P0[a * 64 + i];
                s[a] = (i < 16 * (J + 1)) ? P1[a * 64 + i] : 0.0;
            }
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int j = 4 * p + a;
                const double piv = lane_value(x[a], j);
                bad |= (piv > 0.0) ? 0 : 1;  // (its point's results are dropped)
                // 1 / sqrt(piv): the hardware estimate and two Newton steps,
                // y <- y (3/2 - (piv/2) y^2), and 1 / piv as its square
                const double h = 0.5 * piv;
                double y = __builtin_amdgcn_rsq(piv);
                y = y * fma(-h * y, y, 1.5);
                y = y * fma(-h * y, y, 1.5);
                inv[a] = y * y;
                const double m = (i > j) ? x[a] * inv[a] : 0.0;
                w[a] = s[a] * y;
                nm[a] = -(w[a] * y);
#pragma unroll
                for (int k = a + 1; k < 4; ++k) {
                    const double akj = lane_value(x[a], 4 * p + k);
                    x[k] = fma(-m, akj, x[k]);
                    s[k] = fma(nm[a], akj, s[k]);
                }
            }
            // operands of the tiles, panel column g: of A at row (column) 16 I + c,
            // of S at column 16 I + c
            wave_lds_sync();
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                P0[a * 64 + i] = x[a];
                P1[a * 64 + i] = nm[a];
            }
            wave_lds_sync();
            const double ig = g == 0 ? inv[0] : (g == 1 ? inv[1] : (g == 2 ? inv[2] : inv[3]));
            double u[T], m[T], b[T];
            static_for<J, T>([&](auto Ic) {
                constexpr int I = decltype(Ic)::value;
                u[I] = P0[g * 64 + 16 * I + c];
                m[I] = -(u[I] * ig);
                if constexpr (I == J) m[I] = (16 * J + c > 4 * p + g) ? m[I] : 0.0;
            });
            static_for<0, J + 1>([&](auto Ic) {
                constexpr int I = decltype(Ic)::value;
                b[I] = P1[g * 64 + 16 * I + c];
            });
            // the next panel's columns and rows first; tile column (row) J is done
            // after its fourth panel
            constexpr int J1 = J + (pp == 3 ? 1 : 0);
            static_for<J1, T>([&](auto Kc) {
                constexpr int K = decltype(Kc)::value;
                static_for<K, T>([&](auto Ic) {
                    constexpr int I = decltype(Ic)::value;
                    A[I][K] = __builtin_amdgcn_mfma_f64_16x16x4f64(m[I], u[K], A[I][K], 0, 0, 0);
                });
                static_for<0, J + 1>([&](auto Ic) {
                    constexpr int I = decltype(Ic)::value;
                    S[K][I] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[K], b[I], S[K][I], 0, 0, 0);
                });
            });
            // W_q's rows into LDS, packed (those past N, behind the rest, are not read)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int r = 4 * p + a;
                if (i <= r) Lc[r * (r + 1) / 2 + i] = w[a];
            }
        });
        if (q + gridDim.x < G && i < N) s_next = S64[(q + gridDim.x) * N + i];
        wave_lds_sync();
        if (bad) {  // uniform; the build fails as a whole
            if (i == 0) atomicMin(bad_q, (unsigned long long)q);
            continue;
        }
        double *const sdl = P0, *const sdo = P1;
        sdl[i] = si - (double)(float)si;  // S_q - fl32(S_q)
        sdo[i] = si - off_i;              // S_q - o
        wave_lds_sync();

        // ---- W_q: the packed rows to HBM -----------------------------------------
        if (forms & FC_FORM_FP64) {
            const int nt = N * (N + 1) / 2;
            double *Wq = W64 + q * nt;
            constexpr int B = 13;  // stores prepared at a time
            for (int e0 = i; e0 < nt; e0 += 64 * B) {
                double v[B];
#pragma unroll
                for (int k = 0; k < B; ++k) v[k] = Lc[e0 + 64 * k < nt ? e0 + 64 * k : 0];
#pragma unroll
                for (int k = 0; k < B; ++k)
                    if (e0 + 64 * k < nt) Wq[e0 + 64 * k] = v[k];
            }
        }
        // ---- the requested record forms ----------------------------------------
        if (forms & FC_FORM_FP64) {
            CovEntries<2> m64[cov_units64(NP)];
            cov_entries(map64, f64_rec_units(N), i, m64);
            cov_records(m64, f64_rec_units(N), Lc, cov_region(NP), i,
                        R64 + q * (int64_t)f64_rec_units(N), [](const double (&v)[2]) {
                            return __builtin_bit_cast(uint4, make_double2(v[0], v[1]));
                        });
        }
        if (forms & FC_FORM_FP32) {
            uint4 *rq = R32 + q * (int64_t)rec_units(ns);
            CovEntries<4> m32[cov_units32(NP)];
            cov_entries(map32, rec_w_units(ns), i, m32);
            cov_records(m32, rec_w_units(ns), Lc, cov_region(NP), i, rq,
                        [](const double (&v)[4]) {
                            return __builtin_bit_cast(uint4,
                                                      make_float4((float)v[0], (float)v[1],
                                                                  (float)v[2], (float)v[3]));
                        });
            // FP32 part of the signal (real bin order), then minus W_q times
            // its rounding error (padded row order)
            float *Sp = reinterpret_cast<float *>(rq + rec_w_units(ns));
            Sp[i] = (i < N) ? (float)si : 0.0f;
            const int rr = i - fp32_pad(ns, N);
            double cv = 0.0;
            if (rr >= 0 && rr < N) {
                const double *wr = Lc + rr * (rr + 1) / 2;
#pragma unroll 8
                for (int kk = 0; kk <= rr; ++kk) cv -= wr[kk] * sdl[kk];
            }
            Sp[64 + i] = (float)cv;
        }
        if (forms & (FC_FORM_SPLIT_BF16 | FC_FORM_SPLIT_FP16)) {
            CovEntries<8> m16[cov_units16(NP)];
            cov_entries(map16, code_nfrag(split_code(N)) * 64, i, m16);
            double wmax = 0.0;  // FP16's scale
            if (forms & FC_FORM_SPLIT_FP16) {
                for (int e = i; e < N * (N + 1) / 2; e += 64) wmax = fmax(wmax, fabs(Lc[e]));
                for (int m = 32; m > 0; m >>= 1) wmax = fmax(wmax, __shfl_xor(wmax, m));
            }
            const int64_t sru = split_rec_units(N);
            if (forms & FC_FORM_SPLIT_BF16)
                write_split_record<false>(Lc, sdo, m16, N, 0, wmax, RB16 + q * sru, i);
            if (forms & FC_FORM_SPLIT_FP16)
                write_split_record<true>(Lc, sdo, m16, N, ed16, wmax, RH16 + q * sru, i);
        }
        wave_lds_sync();  // before the next point's LDS writes
    }
}

template <int NP>
hipError_t launch_cov_np(const fc_grid *g, const double *F, const double *stat,
                                int stat_mode, uint32_t forms, const int16_t *maps, double *W64,
                                uint4 *R64, uint4 *R32, uint4 *RB16, uint4 *RH16,
                                unsigned long long *bad_q, hipStream_t st)
{
    const int64_t blocks = g->G < 65536 ? g->G : 65536;
    ProfScope prof(st, "k_cov_build");
    hipLaunchKernelGGL(k_cov_build<NP>, dim3((unsigned)blocks), dim3(64),
                       sizeof(double) * cov_lds_doubles(NP), st, g->S64, F, stat, g->off, g->N,
                       g->G, stat_mode, forms, g->ns, g->ed16, maps, W64, R64, R32, RB16, RH16,
                       bad_q);
    return hipGetLastError();
}

}  // namespace fcx
