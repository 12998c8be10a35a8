// Dispatch of an evolve launch to its kernels: Monte-Carlo sums (evolve_mc2.hip, evolve_mc3.hip), the
// image-gradient centre force and the exact lattice sums (evolve_options.hip). The per-contour code they
// share is in evolve_core.h.
#include "evolve_core.h"

namespace snk {

hipError_t launch_evolve(const EvolveArgs &a, int dim, int lanes, int unroll, int layout, bool trace,
                         hipStream_t s) {
    if (a.n <= 0 || a.n_iter <= 0) return hipSuccess;
    if (a.p.flags & kFlagGradI) {
        if (a.p.flags & kFlagExact) return hipErrorInvalidValue;
        return launch_evolve_gradi(a, dim, lanes, layout, trace, s);
    }
    if (a.p.flags & kFlagExact) {
        if (layout == kBufferQuad) return hipErrorInvalidValue;
        return launch_evolve_exact(a, dim, lanes, layout, trace, s);
    }
    return dim == 2 ? launch_evolve_mc2(a, lanes, unroll, layout, trace, s)
                    : launch_evolve_mc3(a, lanes, unroll, layout, trace, s);
}

int evolve_stage_blocks_per_cu(int dim, int lanes, int unroll, int layout) {
    if (layout != kBufferQuad && layout != kBufferPlain && layout != kBufferPair) return 0;
    return dim == 2 ? evolve_stage_blocks2(lanes, unroll, layout) : evolve_stage_blocks3(lanes, unroll, layout);
}

size_t evolve_lds_bytes(int dim, int lanes, int M, int tile_cap, bool two_waves) {
    const int MH = M / 2;
    if (lanes < 64) return sizeof(float) * (size_t)(64 / lanes * ((draw_floats(lanes, MH) + 3) & ~3));
    const DrawPlan d = draw_plan(dim, MH, tile_cap > 0);
    return wave_lds_bytes(lanes, two_waves ? 128 : lanes, wave_draw_floats(dim, d.K, d.KR, MH), tile_cap);
}

size_t evolve_rule_lds(int dim, int lanes, int M) {
    const int per = (draw_floats(lanes, M / 2) + 3) & ~3;
    const int cpb = lanes < 64 ? 64 / lanes : 1;
    return sizeof(float) * ((size_t)cpb * per + (lanes > 64 ? 2 * (2 + dim) * (lanes / 64) : 0));
}

bool evolve_lds_accepts(int dim, int lanes, int M, int tile_cap) {
    return evolve_rule_lds(dim, lanes, M) + sizeof(float) * (size_t)tile_cap <= 65536;
}

}  // namespace snk
