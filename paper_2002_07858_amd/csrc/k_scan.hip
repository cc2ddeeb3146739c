// k_scan.hip -- the FP32 scan in the residual form (k_scan_fp32.h), and the start
// and the end of the running minima.
#include "k_scan_fp32.h"

namespace fcx {

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
int resident_slots(const void *kernel, int block_threads, size_t dynamic_lds)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
        return 512;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block_threads, dynamic_lds) !=
            hipSuccess ||
        per_cu <= 0)
        per_cu = 2;
    return cus * per_cu;
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
    const ScanGeometry sg = scan_geometry(tiles, tiles, nq, slots, nq, kFp32Chunks);
    const int64_t blocks = sg.n_utiles * sg.n_qchunks;
    ProfScope prof(st, "k_scan_fp32");
    hipLaunchKernelGGL((k_scan_fp32<N>), dim3((unsigned)blocks), dim3(64 * kWavesPerBlock), 0, st,
                       g->R32, d, p_idx, K, q0, q0 + nq, sg.n_utiles, sg.q_per_chunk, keys, chi2_p);
    return hipGetLastError();
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
