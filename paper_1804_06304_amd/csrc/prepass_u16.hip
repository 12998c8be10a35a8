// Pre-pass kernels of u16 volumes.
#include "prepass_core.h"

namespace snk {

hipError_t launch_prepass_u16(const PrepassJob &one, const PrepassJob *jobs, int n, int blocks, hipStream_t s, int *slots) {
    return launch_r<uint16_t>(one, jobs, n, blocks, s, slots);
}

}  // namespace snk
