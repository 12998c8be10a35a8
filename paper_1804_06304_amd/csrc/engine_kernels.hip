// Small kernels of the batch / serving engine. They replace memset and memcpy nodes so that a whole
// batched run can be captured in one hipGraph and replayed.
#include <algorithm>

#include "snk_internal.h"

namespace snk {

namespace {

// Restore every item's contour state from its job's initial state (start of a batched run).
__global__ void reset_items_kernel(const JobDev *jobs, const int2 *items, int n_items, const DevContour *const *init) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_items) return;
    const int2 it = items[i];
    jobs[it.x].st[it.y] = init[it.x][it.y];
}

__global__ void zero_kernel(unsigned long long *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// Per job: whether a contour can still evolve (ACTIVE and below the job's iteration target). Every one that can
// stores the same 1; counting them by atomics on a word per job took 23 us for ten tiles.
__global__ void mark_unfinished_kernel(const JobDev *jobs, const int2 *items, int n_items, int *unfinished) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_items) return;
    const int2 it = items[i];
    const DevContour &c = jobs[it.x].st[it.y];
    if ((c.status & 0x0f) == SNK_ACTIVE && c.iters < jobs[it.x].target) unfinished[it.x] = 1;
}

// One workgroup per piece of at most 16 KB.
__global__ __launch_bounds__(256) void spread_kernel(const char *stage, int n) {
    const CopyPiece p = reinterpret_cast<const CopyPiece *>(stage)[blockIdx.x];
    const uint32_t *src = reinterpret_cast<const uint32_t *>(stage + sizeof(CopyPiece) * (size_t)n + p.at);
    uint32_t *dst = static_cast<uint32_t *>(p.dst);
    for (unsigned i = threadIdx.x; i < p.bytes / 4; i += 256) dst[i] = src[i];
}

__global__ __launch_bounds__(256) void gather_kernel(const JobDev *jobs, const int2 *items, int n_items,
                                                     const unsigned long long *counter, char *out) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0) *reinterpret_cast<unsigned long long *>(out) = *counter;
    if (i >= n_items) return;
    const int2 it = items[i];
    reinterpret_cast<DevContour *>(out + 16)[i] = jobs[it.x].st[it.y];
}

}  // namespace

hipError_t launch_spread(const void *stage, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(spread_kernel, dim3(n), dim3(256), 0, s, static_cast<const char *>(stage), n);
    return hipGetLastError();
}

hipError_t launch_gather(const JobDev *jobs, const int2 *items, int n_items, const unsigned long long *counter, void *out,
                         hipStream_t s) {
    hipLaunchKernelGGL(gather_kernel, dim3(std::max(1, (n_items + 255) / 256)), dim3(256), 0, s, jobs, items, n_items,
                       counter, static_cast<char *>(out));
    return hipGetLastError();
}

hipError_t launch_reset_items(const JobDev *jobs, const int2 *items, int n_items, const DevContour *const *init,
                              hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    hipLaunchKernelGGL(reset_items_kernel, dim3((n_items + 255) / 256), dim3(256), 0, s, jobs, items, n_items, init);
    return hipGetLastError();
}

hipError_t launch_zero(unsigned long long *p, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_mark_unfinished(const JobDev *jobs, const int2 *items, int n_items, int *unfinished, hipStream_t s) {
    if (n_items <= 0) return hipSuccess;
    hipLaunchKernelGGL(mark_unfinished_kernel, dim3((n_items + 255) / 256), dim3(256), 0, s, jobs, items, n_items,
                       unfinished);
    return hipGetLastError();
}

}  // namespace snk
