// Batched evolution over (job, contour) items of many volumes.
#include "evolve_core.h"

namespace snk {

namespace {

// Batched launch over (job, contour) items, one workgroup (G >= 64 lanes) per item. PERSISTENT: a
// fixed grid pops items from a device work queue until it is exhausted (every workgroup reaches
// the exit); otherwise one workgroup per item. STAGE: the workgroup's LDS ends with a box of
// a.tile_cap voxels for the contour it is running (restaged for each item).
// FULL: L = 16 and whole passes (full_passes).
template <int DIM, int G, int U, int LAYOUT, bool PERSISTENT, bool STAGE, bool FULL>
__global__ __launch_bounds__(G, (waves_asked<DIM, G, U, LAYOUT, STAGE, false, FULL>())) void evolve_batch_kernel(BatchArgs a) {
    static_assert(G >= 64, "batched groups span whole waves");
    extern __shared__ __align__(16) float lds[];
    __shared__ int item_sh;
    for (int round = 0;; ++round) {
        int item;
        if constexpr (PERSISTENT) {
            if (threadIdx.x == 0) item_sh = atomicAdd(a.queue, 1);
            __syncthreads();
            item = __builtin_amdgcn_readfirstlane(item_sh);
            __syncthreads();
        } else {
            item = round == 0 ? (int)blockIdx.x : a.n_items;
        }
        if (item >= a.n_items) break;
        const int job = __builtin_amdgcn_readfirstlane(a.items[item].x);
        const int cid = __builtin_amdgcn_readfirstlane(a.items[item].y);
        const JobParams p = uniform_copy(&a.jobs[job].p);
        DevContour *st = uniform_copy(&a.jobs[job].st);
        const int target = __builtin_amdgcn_readfirstlane(a.jobs[job].target);
        run_wave<DIM, G, U, false, LAYOUT, false, STAGE, false, FULL>(
            p, (Cold<JobParams>)&a.jobs[job].p, st + cid, a.chunk, target, nullptr, lds, a.draw_k, a.rot_k, a.counter,
            STAGE ? a.tile_cap : 0, Repel{nullptr, 0, -1});
        __syncthreads();
    }
}

template <int DIM, int G, int U, int LAYOUT, bool PERSISTENT, bool STAGE>
hipError_t batch_t(BatchArgs a, int grid, hipStream_t s) {
    const int g = PERSISTENT ? grid : a.n_items;
    if (g <= 0) return hipSuccess;
    const DrawPlan d = draw_plan(DIM, a.max_M / 2, STAGE);
    a.draw_k = d.K;
    a.rot_k = d.KR;
    const size_t lds = wave_lds_bytes(G, G, wave_draw_floats(DIM, d.K, d.KR, a.max_M / 2), STAGE ? a.tile_cap : 0);
    if constexpr (U >= 2)
        if (full_passes(G, U, a.max_M, a.L)) {
            hipLaunchKernelGGL((evolve_batch_kernel<DIM, G, U, LAYOUT, PERSISTENT, STAGE, true>), dim3(g), dim3(G), lds,
                               s, a);
            return hipGetLastError();
        }
    hipLaunchKernelGGL((evolve_batch_kernel<DIM, G, U, LAYOUT, PERSISTENT, STAGE, false>), dim3(g), dim3(G), lds, s, a);
    return hipGetLastError();
}

template <int DIM, int G, int U, int LAYOUT, bool PERSISTENT>
hipError_t batch_s(const BatchArgs &a, int grid, hipStream_t s) {
    return a.tile_cap > 0 ? batch_t<DIM, G, U, LAYOUT, PERSISTENT, true>(a, grid, s)
                          : batch_t<DIM, G, U, LAYOUT, PERSISTENT, false>(a, grid, s);
}

template <int DIM, int G, int U, int LAYOUT>
hipError_t batch_p(const BatchArgs &a, bool persistent, int grid, hipStream_t s) {
    return persistent ? batch_s<DIM, G, U, LAYOUT, true>(a, grid, s) : batch_s<DIM, G, U, LAYOUT, false>(a, grid, s);
}

template <int DIM, int G, int U>
hipError_t batch_l(const BatchArgs &a, int layout, bool persistent, int grid, hipStream_t s) {
    if (layout == kBufferPair) return batch_p<DIM, G, U, kBufferPair>(a, persistent, grid, s);
    return layout == kBufferQuad ? batch_p<DIM, G, U, kBufferQuad>(a, persistent, grid, s)
                                 : batch_p<DIM, G, U, kBufferPlain>(a, persistent, grid, s);
}

template <int DIM, int G>
hipError_t batch_u(const BatchArgs &a, int unroll, int layout, bool persistent, int grid, hipStream_t s) {
    return unroll >= 2 ? batch_l<DIM, G, 2>(a, layout, persistent, grid, s)
                       : batch_l<DIM, G, 1>(a, layout, persistent, grid, s);
}

template <int DIM>
hipError_t batch_g(const BatchArgs &a, int lanes, int unroll, int layout, bool persistent, int grid,
                   hipStream_t s) {
    switch (lanes) {
        case 64: return batch_u<DIM, 64>(a, unroll, layout, persistent, grid, s);
        case 128: return batch_u<DIM, 128>(a, unroll, layout, persistent, grid, s);
        default: return batch_u<DIM, 256>(a, unroll, layout, persistent, grid, s);
    }
}

// Workgroups per CU of the general instance (a FULL one needs no more registers).
template <int DIM, int G, int U, int LAYOUT, bool STAGE>
int max_blocks_t(int max_M, int tile_cap) {
    int blocks = 0;
    const size_t lds = evolve_lds_bytes(DIM, G, max_M, STAGE ? tile_cap : 0);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &blocks, evolve_batch_kernel<DIM, G, U, LAYOUT, true, STAGE, false>, G, lds) != hipSuccess)
        return 1;
    return blocks > 0 ? blocks : 1;
}

template <int DIM, int G, int U, int LAYOUT>
int max_blocks_s(int max_M, int tile_cap) {
    return tile_cap > 0 ? max_blocks_t<DIM, G, U, LAYOUT, true>(max_M, tile_cap)
                        : max_blocks_t<DIM, G, U, LAYOUT, false>(max_M, 0);
}

template <int DIM, int G>
int max_blocks_u(int unroll, int layout, int max_M, int tile_cap) {
    if (unroll >= 2) {
        if (layout == kBufferPair) return max_blocks_s<DIM, G, 2, kBufferPair>(max_M, tile_cap);
        return layout == kBufferQuad ? max_blocks_s<DIM, G, 2, kBufferQuad>(max_M, tile_cap)
                                     : max_blocks_s<DIM, G, 2, kBufferPlain>(max_M, tile_cap);
    }
    if (layout == kBufferPair) return max_blocks_s<DIM, G, 1, kBufferPair>(max_M, tile_cap);
    return layout == kBufferQuad ? max_blocks_s<DIM, G, 1, kBufferQuad>(max_M, tile_cap)
                                 : max_blocks_s<DIM, G, 1, kBufferPlain>(max_M, tile_cap);
}

template <int DIM>
int max_blocks_g(int lanes, int unroll, int layout, int max_M, int tile_cap) {
    switch (lanes) {
        case 64: return max_blocks_u<DIM, 64>(unroll, layout, max_M, tile_cap);
        case 128: return max_blocks_u<DIM, 128>(unroll, layout, max_M, tile_cap);
        default: return max_blocks_u<DIM, 256>(unroll, layout, max_M, tile_cap);
    }
}

}  // namespace

hipError_t launch_evolve_batch(const BatchArgs &a, int dim, int lanes, int unroll, int layout, bool persistent,
                               int grid, hipStream_t s) {
    if (a.n_items <= 0 || a.chunk <= 0) return hipSuccess;
    if (layout != kBufferQuad && layout != kBufferPlain && layout != kBufferPair) return hipErrorInvalidValue;
    if (dim == 2) return batch_g<2>(a, lanes, unroll, layout, persistent, grid, s);
    return batch_g<3>(a, lanes, unroll, layout, persistent, grid, s);
}

int evolve_batch_max_blocks(int dim, int lanes, int unroll, int layout, int max_M, int tile_cap) {
    return dim == 2 ? max_blocks_g<2>(lanes, unroll, layout, max_M, tile_cap)
                    : max_blocks_g<3>(lanes, unroll, layout, max_M, tile_cap);
}

}  // namespace snk
