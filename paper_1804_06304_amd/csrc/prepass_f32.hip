// Pre-pass kernels of f32 volumes.
#include "prepass_core.h"

namespace snk {

hipError_t launch_prepass_f32(const PrepassJob &one, const PrepassJob *jobs, int n, int blocks, hipStream_t s, int *slots) {
    return launch_r<float>(one, jobs, n, blocks, s, slots);
}

}  // namespace snk
