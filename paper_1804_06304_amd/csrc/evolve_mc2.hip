// Monte-Carlo evolution kernels, dim 2.
#include "evolve_mc.h"

namespace snk {

hipError_t launch_evolve_mc2(const EvolveArgs &a, int lanes, int unroll, int layout, bool trace, hipStream_t s) {
    return trace ? launch_g<2, true>(a, lanes, unroll, layout, s) : launch_g<2, false>(a, lanes, unroll, layout, s);
}

int evolve_stage_blocks2(int lanes, int unroll, int layout) { return stage_blocks_g<2>(lanes, unroll, layout); }

}  // namespace snk
