// Evolution kernels of the options: the image-gradient centre force and the exact lattice sums.
#include "evolve_core.h"

namespace snk {

namespace {

// Gradient-form centre force: whole-wave groups, two pair-points in flight, buffer layouts, with or
// without LDS boxes.
template <int DIM, int G, bool TRACE>
hipError_t launch_gradi_l(const EvolveArgs &a, int layout, hipStream_t s) {
    const bool stage = a.tile_cap > 0;
    if (layout == kBufferQuad)
        return stage ? launch_t<DIM, G, 2, TRACE, kBufferQuad, false, true, true>(a, s)
                     : launch_t<DIM, G, 2, TRACE, kBufferQuad, false, false, true>(a, s);
    if (layout == kBufferPlain)
        return stage ? launch_t<DIM, G, 2, TRACE, kBufferPlain, false, true, true>(a, s)
                     : launch_t<DIM, G, 2, TRACE, kBufferPlain, false, false, true>(a, s);
    if constexpr (DIM == 3)
        if (layout == kBufferPair)
            return stage ? launch_t<DIM, G, 2, TRACE, kBufferPair, false, true, true>(a, s)
                         : launch_t<DIM, G, 2, TRACE, kBufferPair, false, false, true>(a, s);
    return hipErrorInvalidValue;
}

template <int DIM, bool TRACE>
hipError_t launch_gradi_g(const EvolveArgs &a, int lanes, int layout, hipStream_t s) {
    switch (lanes) {
        case 64: return launch_gradi_l<DIM, 64, TRACE>(a, layout, s);
        case 128: return launch_gradi_l<DIM, 128, TRACE>(a, layout, s);
        case 256: return launch_gradi_l<DIM, 256, TRACE>(a, layout, s);
        default: return hipErrorInvalidValue;
    }
}

// Exact lattice sums read single voxels: plain layouts only.
template <int DIM, int G, bool TRACE>
hipError_t launch_exact_l(const EvolveArgs &a, int layout, hipStream_t s) {
    return layout == kGlobalPlain ? launch_t<DIM, G, 1, TRACE, kGlobalPlain, true>(a, s)
                                  : launch_t<DIM, G, 1, TRACE, kBufferPlain, true>(a, s);
}

template <int DIM, bool TRACE>
hipError_t launch_exact_g(const EvolveArgs &a, int lanes, int layout, hipStream_t s) {
    switch (lanes) {
        case 16: return launch_exact_l<DIM, 16, TRACE>(a, layout, s);
        case 32: return launch_exact_l<DIM, 32, TRACE>(a, layout, s);
        case 64: return launch_exact_l<DIM, 64, TRACE>(a, layout, s);
        case 128: return launch_exact_l<DIM, 128, TRACE>(a, layout, s);
        default: return launch_exact_l<DIM, 256, TRACE>(a, layout, s);
    }
}

}  // namespace

hipError_t launch_evolve_gradi(const EvolveArgs &a, int dim, int lanes, int layout, bool trace, hipStream_t s) {
    if (dim == 2) return trace ? launch_gradi_g<2, true>(a, lanes, layout, s) : launch_gradi_g<2, false>(a, lanes, layout, s);
    return trace ? launch_gradi_g<3, true>(a, lanes, layout, s) : launch_gradi_g<3, false>(a, lanes, layout, s);
}

hipError_t launch_evolve_exact(const EvolveArgs &a, int dim, int lanes, int layout, bool trace, hipStream_t s) {
    if (dim == 2) return trace ? launch_exact_g<2, true>(a, lanes, layout, s) : launch_exact_g<2, false>(a, lanes, layout, s);
    return trace ? launch_exact_g<3, true>(a, lanes, layout, s) : launch_exact_g<3, false>(a, lanes, layout, s);
}

}  // namespace snk
