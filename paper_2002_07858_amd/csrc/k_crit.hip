// k_crit.hip -- critical values and histogram of Delta chi^2 per true point.
//
// Section 1 / Figure 1: the critical value for a fraction alpha is the value
// left of which that fraction of the Delta chi^2 distribution lies.  It is
// taken as the type-1 order statistic x_(j), j = ceil(alpha K) clamped to
// [1, K], with NaN ordered last.  One block per segment finds x_(j) for every
// alpha over 64-bit keys whose unsigned order is the numeric order of the
// doubles: the keys between the segment's smallest and largest are counted in
// 2^BITS equal intervals, each rank's interval is cut again until it holds at
// most kCand keys (one or two cuts: the intervals of the first already split
// the range the values occupy, where a fixed radix spends its first digits on
// the sign and exponent they share and its counters on one address), and those
// are ranked directly.  No sort, no scratch memory beyond LDS; the first
// KR T keys stay in registers between the passes.
//
// Bound: latency of one block (loads, LDS atomics, a barrier per pass).  With
// three alphas and a 200-bin histogram, one segment of 1000 / 5000 / 20 000
// values takes 11 / 23 / 45 us; the 8-pass radix select of 256 threads that
// this replaced took 23 / 89 / 273 us.
#include "fc_internal.h"

namespace fcx {

constexpr int kMaxAlpha = 8;

struct AlphaArgs {
    double a[kMaxAlpha];
};

__device__ __forceinline__ unsigned long long order_key(double x)
{
    if (x != x) return ~0ull;  // NaN sorts last
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ __forceinline__ double from_order_key(unsigned long long k)
{
    if (k == ~0ull) return __builtin_nan("");
    const unsigned long long b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
    return __longlong_as_double((long long)b);
}

constexpr int kCand = 256;  // keys ranked directly

// Segment s is x[seg_lo[s] .. seg_hi[s]).  The order statistics taken are
// ranks ceil(alpha K) (alpha mode), or ranks[s][a] (1-based, clamped to
// [1, K]) when a rank table is given.
template <int T, int BITS, int KR>
__global__ __launch_bounds__(T) void k_crit(const int64_t *__restrict__ seg_lo,
                                            const int64_t *__restrict__ seg_hi,
                                            const double *__restrict__ x, int n_alpha,
                                            AlphaArgs alpha, const int64_t *__restrict__ ranks,
                                            double *__restrict__ crit, int n_bins, double hist_hi,
                                            int64_t *__restrict__ hist)
{
    constexpr int BINS = 1 << BITS, NW = T / 64;
    static_assert(T % kCand == 0 && BINS % 64 == 0 && kMaxAlpha * BINS * 4 >= kMaxAlpha * kCand * 8, "LDS sharing");
    // counters of every rank's interval, then its remaining keys
    __shared__ union {
        unsigned int cnt[kMaxAlpha][BINS];
        unsigned long long cand[kMaxAlpha][kCand];
    } sh;
    __shared__ unsigned long long lo_s[kMaxAlpha], red[2][NW];
    __shared__ long long rank_s[kMaxAlpha];
    __shared__ unsigned int num_s[kMaxAlpha], fill_s[kMaxAlpha];
    __shared__ int shift_s[kMaxAlpha];
    extern __shared__ unsigned int hbin[];

    const int64_t sgi = blockIdx.x;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int64_t lo = seg_lo[sgi], hi = seg_hi[sgi];
    const bool valid = lo >= 0 && hi >= lo;
    const int64_t K = valid ? hi - lo : 0;

    if (hist) {
        for (int b = tid; b <= n_bins; b += T) hbin[b] = 0u;
        __syncthreads();
    }
    const double width = hist ? hist_hi / (double)n_bins : 1.0;
    const auto count = [&](double v) {
        int b = n_bins;
        if (v >= 0.0 && v < hist_hi) {
            const double f = floor(v / width);
            b = (f > (double)(n_bins - 1)) ? n_bins - 1 : (int)f;
        }
        atomicAdd(&hbin[b], 1u);
    };
    // one pass over the values: histogram, smallest and largest key
    unsigned long long key[KR], kmin = ~0ull, kmax = 0ull;
    const auto first = [&](double v) {
        if (hist) count(v);
        const unsigned long long k = order_key(v);
        kmin = k < kmin ? k : kmin;
        kmax = k > kmax ? k : kmax;
        return k;
    };
    if (K > 0) {
        double v[KR];  // the loads first (clamped to the segment), then their use
#pragma unroll
        for (int i = 0; i < KR; ++i)
            if ((int64_t)i * T < K) v[i] = x[lo + (i * T + tid < K ? i * T + tid : K - 1)];
#pragma unroll
        for (int i = 0; i < KR; ++i)
            if (i * T + tid < K) key[i] = first(v[i]);
    }
    for (int64_t k = (int64_t)KR * T + tid; k < K; k += T) (void)first(x[lo + k]);
    // later passes: fn(key) for every key of the segment
    const auto each = [&](auto fn) {
#pragma unroll
        for (int i = 0; i < KR; ++i)
            if (i * T + tid < K) fn(key[i]);
        for (int64_t k = (int64_t)KR * T + tid; k < K; k += T) fn(order_key(x[lo + k]));
    };
    if (K == 0) {
        if (hist)
            for (int b = tid; b <= n_bins; b += T) hist[sgi * (int64_t)(n_bins + 1) + b] = 0;
        if (tid < n_alpha) crit[sgi * n_alpha + tid] = __builtin_nan("");
        return;
    }
    for (int m = 32; m > 0; m >>= 1) {
        const unsigned long long a = __shfl_xor(kmin, m), b = __shfl_xor(kmax, m);
        kmin = a < kmin ? a : kmin;
        kmax = b > kmax ? b : kmax;
    }
    if (lane == 0) {
        red[0][wave] = kmin;
        red[1][wave] = kmax;
    }
    for (int e = tid; e < BINS; e += T) sh.cnt[0][e] = 0u;
    __syncthreads();
    if (hist)
        for (int b = tid; b <= n_bins; b += T)
            hist[sgi * (int64_t)(n_bins + 1) + b] = (int64_t)hbin[b];
    for (int w = 0; w < NW; ++w) {
        kmin = red[0][w] < kmin ? red[0][w] : kmin;
        kmax = red[1][w] > kmax ? red[1][w] : kmax;
    }
    // 2^s keys an interval, the fewest that leave 2^BITS intervals
    const unsigned long long span = kmax - kmin;
    const int s0 = (span >> BITS) ? 64 - BITS - __builtin_clzll(span) : 0;
    if (tid < n_alpha) {
        long long j = ranks ? (long long)ranks[sgi * n_alpha + tid]
                            : (long long)ceil(alpha.a[tid] * (double)K);
        if (j < 1) j = 1;
        if (j > K) j = K;
        rank_s[tid] = j - 1;  // 0-based
        lo_s[tid] = kmin;
        shift_s[tid] = s0;
        num_s[tid] = (unsigned int)K;
        fill_s[tid] = 0u;
    }
    // interval of rank rank_s[a] in table t: wave a, lane l holding bins
    // l BINS/64 ..., a prefix sum over the lanes finds the lane that covers it
    const auto pick = [&](int a, int t, int s) {  // table t's intervals: 2^s keys each
        constexpr int PER = BINS / 64;
        const long long r = rank_s[a];
        long long own = 0;
        for (int e = 0; e < PER; ++e) own += sh.cnt[t][lane * PER + e];
        long long incl = own;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const long long up = __shfl_up(incl, off, 64);
            if (lane >= off) incl += up;
        }
        if (incl - own <= r && r < incl) {
            long long rr = r - (incl - own);
            int e = lane * PER;
            while (rr >= sh.cnt[t][e]) rr -= sh.cnt[t][e++];
            rank_s[a] = rr;
            num_s[a] = sh.cnt[t][e];
            lo_s[a] += (unsigned long long)e << s;
            shift_s[a] = s;
        }
    };
    if (K > kCand) {
        // the first cut is the same for every rank
        each([&](unsigned long long k) { atomicAdd(&sh.cnt[0][(k - kmin) >> s0], 1u); });
        __syncthreads();
        for (int a = wave; a < n_alpha; a += NW) pick(a, 0, s0);
        for (;;) {
            __syncthreads();
            bool more = false;
            for (int a = 0; a < n_alpha; ++a)
                more = more || (shift_s[a] > 0 && num_s[a] > (unsigned)kCand);
            if (!more) break;  // uniform
            for (int e = tid; e < n_alpha * BINS; e += T) (&sh.cnt[0][0])[e] = 0u;
            __syncthreads();
            each([&](unsigned long long k) {
                for (int a = 0; a < n_alpha; ++a) {
                    const int s = shift_s[a];
                    if (s > 0 && num_s[a] > (unsigned)kCand && k >= lo_s[a] &&
                        ((k - lo_s[a]) >> s) == 0)
                        atomicAdd(&sh.cnt[a][(k - lo_s[a]) >> (s > BITS ? s - BITS : 0)], 1u);
                }
            });
            __syncthreads();
            for (int a = wave; a < n_alpha; a += NW)
                if (shift_s[a] > 0 && num_s[a] > (unsigned)kCand)
                    pick(a, a, shift_s[a] > BITS ? shift_s[a] - BITS : 0);
        }
    }
    __syncthreads();
    // keys below list[i] among its first n, equal ones by position; SUB lanes
    // share a key's comparisons, so that a wide block is not mostly idle
    constexpr int SUB = T / kCand;
    const auto below = [&](const unsigned long long *list, int n, int i) {
        const unsigned long long own = list[i];
        int b = 0;
#pragma unroll 8
        for (int c = tid % SUB; c < n; c += SUB)
            b += (list[c] < own || (list[c] == own && c < i)) ? 1 : 0;
#pragma unroll
        for (int m = 1; m < SUB; m <<= 1) b += __shfl_xor(b, m);
        return b;
    };
    if (K <= kCand) {
        // every key's rank, once for all alphas
        each([&](unsigned long long k) { sh.cand[0][atomicAdd(&fill_s[0], 1u)] = k; });
        __syncthreads();
        const int i = tid / SUB;
        if (i < (int)K) {
            const int r = below(sh.cand[0], (int)K, i);
            for (int a = 0; a < n_alpha; ++a)
                if (r == (int)rank_s[a])
                    crit[sgi * n_alpha + a] = from_order_key(sh.cand[0][i]);
        }
        return;
    }
    // the keys of every rank's interval, and the one of that rank among them
    // (an interval of one key value needs none)
    each([&](unsigned long long k) {
        for (int a = 0; a < n_alpha; ++a) {
            const int s = shift_s[a];
            if (s > 0 && k >= lo_s[a] && ((k - lo_s[a]) >> s) == 0)
                sh.cand[a][atomicAdd(&fill_s[a], 1u)] = k;
        }
    });
    __syncthreads();
    if (tid < n_alpha && shift_s[tid] == 0) crit[sgi * n_alpha + tid] = from_order_key(lo_s[tid]);
    // (the intervals' keys one after the other: at a time they are few for the block)
    for (int e = tid / SUB;; e += kCand) {
        int a = 0, i = e;
        while (a < n_alpha && i >= (int)fill_s[a]) i -= (int)fill_s[a++];
        if (a == n_alpha) break;
        if (below(sh.cand[a], (int)fill_s[a], i) == (int)rank_s[a])
            crit[sgi * n_alpha + a] = from_order_key(sh.cand[a][i]);
    }
}

namespace {

// Up to a segment a CU: 1024 threads each, since a block's own latency is the
// time; up to two, 512, so that both are resident; more, 256, so that several
// share a CU.  300 segments of 300 / 2000 / 20 000 values: 1024 threads 20 / 21 /
// 57 us, 512 10 / 13 / 58, 256 11 / 13 / 183; 256 segments of 20 000: 1024 threads
// 31 us, 256 166; 1600 of 2048: 1024 threads 70 us, 256 19.
hipError_t launch_crit_any(int64_t n_seg, const int64_t *seg_lo, const int64_t *seg_hi,
                           const double *x, int n_alpha, const AlphaArgs &aa,
                           const int64_t *ranks, double *crit, int n_bins, double hist_hi,
                           int64_t *hist, hipStream_t st)
{
    const size_t lds = hist ? sizeof(unsigned int) * (size_t)(n_bins + 1) : 0;
    if (n_seg <= 256)
        hipLaunchKernelGGL((k_crit<1024, 10, 20>), dim3((unsigned)n_seg), dim3(1024), lds, st,
                           seg_lo, seg_hi, x, n_alpha, aa, ranks, crit, n_bins, hist_hi, hist);
    else if (n_seg <= 512)
        hipLaunchKernelGGL((k_crit<512, 10, 20>), dim3((unsigned)n_seg), dim3(512), lds, st,
                           seg_lo, seg_hi, x, n_alpha, aa, ranks, crit, n_bins, hist_hi, hist);
    else
        hipLaunchKernelGGL((k_crit<256, 9, 10>), dim3((unsigned)n_seg), dim3(256), lds, st, seg_lo,
                           seg_hi, x, n_alpha, aa, ranks, crit, n_bins, hist_hi, hist);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_crit(int64_t n_seg, const int64_t *seg_off, const double *x, int n_alpha,
                       const double *alpha, double *crit, int n_bins, double hist_hi,
                       int64_t *hist, hipStream_t st)
{
    AlphaArgs aa;
    for (int a = 0; a < kMaxAlpha; ++a) aa.a[a] = (a < n_alpha) ? alpha[a] : 1.0;
    return launch_crit_any(n_seg, seg_off, seg_off + 1, x, n_alpha, aa, nullptr, crit, n_bins,
                           hist_hi, hist, st);
}

hipError_t launch_crit_gapped(int64_t n_seg, const int64_t *seg_lo, const int64_t *seg_hi,
                              const double *x, int n_alpha, const double *alpha, double *crit,
                              hipStream_t st)
{
    AlphaArgs aa;
    for (int a = 0; a < kMaxAlpha; ++a) aa.a[a] = (a < n_alpha) ? alpha[a] : 1.0;
    return launch_crit_any(n_seg, seg_lo, seg_hi, x, n_alpha, aa, nullptr, crit, 0, 1.0, nullptr,
                           st);
}

hipError_t launch_select_ranks(int64_t n_seg, const int64_t *seg_lo, const int64_t *seg_hi,
                               const double *x, int n_q, const int64_t *ranks, double *out,
                               hipStream_t st)
{
    AlphaArgs aa;
    for (int a = 0; a < kMaxAlpha; ++a) aa.a[a] = 1.0;
    return launch_crit_any(n_seg, seg_lo, seg_hi, x, n_q, aa, ranks, out, 0, 1.0, nullptr, st);
}

}  // namespace fcx
