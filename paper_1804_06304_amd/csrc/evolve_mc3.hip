// Monte-Carlo evolution kernels, dim 3.
#include "evolve_mc.h"

namespace snk {

hipError_t launch_evolve_mc3(const EvolveArgs &a, int lanes, int unroll, int layout, bool trace, hipStream_t s) {
    return trace ? launch_g<3, true>(a, lanes, unroll, layout, s) : launch_g<3, false>(a, lanes, unroll, layout, s);
}

int evolve_stage_blocks3(int lanes, int unroll, int layout) { return stage_blocks_g<3>(lanes, unroll, layout); }

}  // namespace snk
