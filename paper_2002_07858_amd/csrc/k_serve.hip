// k_serve.hip -- request serving in the FP32 form (k_scan_fp32.h).
#include "k_scan_fp32.h"

namespace fcx {

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

}  // namespace fcx
