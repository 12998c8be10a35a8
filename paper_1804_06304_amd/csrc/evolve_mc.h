// Launch templates of the Monte-Carlo evolution, instantiated per dimension in evolve_mc2.hip and evolve_mc3.hip.
#pragma once

#include "evolve_core.h"

namespace snk {

namespace {

template <int DIM, int G, int U, bool TRACE>
hipError_t launch_l(const EvolveArgs &a, int layout, hipStream_t s) {
    if constexpr (G >= 64) {
        // LDS boxes, with a buffer layout for the iterations whose ball does not fit
        if (a.tile_cap > 0) {
            if (layout == kBufferQuad) return launch_t<DIM, G, U, TRACE, kBufferQuad, false, true>(a, s);
            if (layout == kBufferPlain) return launch_t<DIM, G, U, TRACE, kBufferPlain, false, true>(a, s);
            if constexpr (DIM == 3)
                if (layout == kBufferPair) return launch_t<DIM, G, U, TRACE, kBufferPair, false, true>(a, s);
            return hipErrorInvalidValue;
        }
    } else {
        if (a.tile_cap > 0) return hipErrorInvalidValue;
    }
    switch (layout) {
        case kBufferPair: return launch_t<DIM, G, U, TRACE, kBufferPair>(a, s);
        case kBufferQuad: return launch_t<DIM, G, U, TRACE, kBufferQuad>(a, s);
        case kBufferPlain: return launch_t<DIM, G, U, TRACE, kBufferPlain>(a, s);
        case kGlobalPlain: return launch_t<DIM, G, U, TRACE, kGlobalPlain>(a, s);
        default: return hipErrorInvalidValue;
    }
}

// Four pair-points in flight: half-wave, one- and two-wave groups, outside the per-iteration trace (there the
// order of a lane's sums is the same as with two, so the trace runs the two-pair-point instance).
template <int DIM, int G, bool TRACE>
hipError_t launch_u(const EvolveArgs &a, int unroll, int layout, hipStream_t s) {
    if constexpr (!TRACE && (G == 32 || G == 64 || G == 128))
        if (unroll >= 4) return launch_l<DIM, G, 4, TRACE>(a, layout, s);
    return unroll >= 2 ? launch_l<DIM, G, 2, TRACE>(a, layout, s) : launch_l<DIM, G, 1, TRACE>(a, layout, s);
}

template <int DIM, bool TRACE>
hipError_t launch_g(const EvolveArgs &a, int lanes, int unroll, int layout, hipStream_t s) {
    switch (lanes) {
        case 16: return launch_u<DIM, 16, TRACE>(a, unroll, layout, s);
        case 32: return launch_u<DIM, 32, TRACE>(a, unroll, layout, s);
        case 64: return launch_u<DIM, 64, TRACE>(a, unroll, layout, s);
        case 128: return launch_u<DIM, 128, TRACE>(a, unroll, layout, s);
        default: return launch_u<DIM, 256, TRACE>(a, unroll, layout, s);
    }
}

template <int DIM, int G, int U>
int stage_blocks_t(int layout) {
    int nb = 0;
    hipError_t e;
    if (layout == kBufferQuad)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, evolve_kernel<DIM, G, U, false, kBufferQuad, false, true, false, false>, Grp<G>::NT, 0);
    else if (DIM == 3 && layout == kBufferPair)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, evolve_kernel<DIM, G, U, false, DIM == 3 ? kBufferPair : kBufferPlain, false, true, false, false>,
            Grp<G>::NT, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &nb, evolve_kernel<DIM, G, U, false, kBufferPlain, false, true, false, false>, Grp<G>::NT, 0);
    return e == hipSuccess ? nb : 0;
}

template <int DIM, int G>
int stage_blocks_u(int unroll, int layout) {
    if constexpr (G == 64 || G == 128)
        if (unroll >= 4) return stage_blocks_t<DIM, G, 4>(layout);
    return unroll >= 2 ? stage_blocks_t<DIM, G, 2>(layout) : stage_blocks_t<DIM, G, 1>(layout);
}

template <int DIM>
int stage_blocks_g(int lanes, int unroll, int layout) {
    switch (lanes) {
        case 64: return stage_blocks_u<DIM, 64>(unroll, layout);
        case 128: return stage_blocks_u<DIM, 128>(unroll, layout);
        case 256: return stage_blocks_u<DIM, 256>(unroll, layout);
        default: return 0;
    }
}

}  // namespace

}  // namespace snk
