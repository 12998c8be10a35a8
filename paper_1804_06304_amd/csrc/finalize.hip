// End of evolution (Results of the paper): exact energy and selection.
//
// Exact energy: one workgroup per contour evaluates Eq. (5) over the lattice points within R + dR/2 of the
// centre (clamp-to-edge values outside the volume), times the voxel measure, divided by (2R)^d. Distance,
// weight and sums in FP64, fixed-order reduction. Contours still ACTIVE become MAXITER here.
//
// Selection. Candidates (CONVERGED or MAXITER, E_vox <= E0) are binned on a uniform grid with cell
// >= rho * r_max, so every overlapping pair (|c' - c''| < rho max(R', R'')) lies in neighbouring cells. A
// candidate is accepted once every overlapping candidate with a smaller (E_vox, id) is rejected, and
// rejected once one of them is accepted; that decides the smallest undecided candidate at every step, so the
// result equals the sequential greedy of the paper's competition (lower energy survives) taken in ascending
// (E_vox, id) order.
// Contours are chained per cell, each candidate's overlapping smaller candidates are listed once, and rounds over
// the lists of those that have any decide the rest: of one volume by grid-wide steps (select_plain), of a batch
// by grid-wide lists and a workgroup per job (launch_select_batch).
#include <math.h>

#include <algorithm>

#include "snk_internal.h"

namespace snk {

namespace {

constexpr int SEL_T = 1024;

// Threads per contour of the exact energy: a 3D ball holds thousands of lattice points, a disk
// hundreds.
template <int DIM>
constexpr int ev_threads() {
    return DIM == 3 ? 256 : 64;
}

// Lanes that share a lattice row: a ball of R = 8 has some 200 rows of up to 18 points, a disk of R = 12 has 25
// rows of up to 25.
template <int DIM>
constexpr int ev_share() {
    return DIM == 3 ? 1 : 2;
}

// Bound by instruction issue (62,500 lattice contours: 1,685 vector instructions per wave with a lane per point of the
// ball's box). So a lane takes one row of the lattice and walks only the points of it inside the ball, about a
// quarter of the box, the row's part of the distance is formed once and the weight takes no division. Four points'
// loads are in flight per lane. Finalize, a lane per point -> now: 62,500 lattice contours 754 -> 330 us, 2,000
// contours 71 -> 48, 40,000 in 2D 143 -> 98, 8 contours 30 -> 21.
// Every point's distance has the bits of a correctly rounded root or is next to them: the hardware's reciprocal root,
// one coupled step for the root and half its reciprocal and one for the root's remainder (P. Markstein, IA-64 and
// Elementary Functions, 2000). With the first step alone, and ramps as slope times r plus an offset, sums that
// cancel were off by up to 9 x 2^-53 of their magnitude; now by 0.6, a lane per point and divisions left 1.8.
template <int DIM>
__device__ void energy_one(const JobParams &p, DevContour *slot, double *e_out, bool finalize = true) {
    constexpr int EV_T = ev_threads<DIM>();
    constexpr int SHARE = ev_share<DIM>();
    constexpr double RHO = DIM == 3 ? 0.79370052598409973738 : 0.70710678118654752440;
    __shared__ double part[EV_T / 64];
    const int t = threadIdx.x;
    const DevContour s = *slot;
    const Geometry &g = p.g;
    const float R = s.R;
    if (!isfinite(R) || !(R > 0.0f) || !(R <= p.r_hi) || (s.status & 0x0f) == SNK_NONFINITE) {
        if (t == 0) {
            *e_out = NAN;
            if (finalize) slot->e_vox = NAN;
        }
        return;
    }
    const float smax = R + 0.5f * p.dR;
    const double R_d = (double)R, dR_d = (double)p.dR, smax_d = R_d + 0.5 * dR_d, smax2 = smax_d * smax_d;
    // S(r) (Sec. II-B). Of a radius below the smallest admissible one (a state set by the caller) the inner ramp reaches
    // into the outer one: the first region in order that holds r counts. Else each ramp, held between its ends, is
    // constant where the other one runs. (rho R has twice the bits: what its rounding leaves is in the ramp's offset.)
    const double ain = RHO * R_d, dr = RHO * dR_d, is = 2.0 / dr, in0 = -is * fma(RHO, R_d, -ain), os = -1.0 / dR_d;
    const double core = ain - 0.5 * dr, ramp = ain + 0.5 * dr, shell = R_d - 0.5 * dR_d;
    const bool disjoint = __builtin_amdgcn_readfirstlane(ramp <= shell);
    // rows within the ball's range (a row or point of the margin has no point inside, or weight 0)
    int lo[3] = {0, 0, 0}, cnt[3] = {1, 1, 1};
#pragma unroll
    for (int i = 1; i < DIM; ++i) {
        const float ext = smax * g.inv_h[i];
        lo[i] = (int)floorf(s.off[i] - ext);
        cnt[i] = (int)ceilf(s.off[i] + ext) - lo[i] + 1;
    }
    const int nn[3] = {g.nx, g.ny, g.nz};
    const int total = cnt[1] * cnt[2] * SHARE;
    const double hx = (double)g.h[0], ox = (double)s.off[0];
    double acc = 0.0;
    for (int q = t; q < total; q += EV_T) {
        const int row = q / SHARE, yy = row % cnt[1], zz = row / cnt[1];
        const double dy = ((double)(lo[1] + yy) - (double)s.off[1]) * (double)g.h[1];
        double dz = 0.0, r2 = dy * dy;
        int z = 0;
        if constexpr (DIM == 3) {
            dz = ((double)(lo[2] + zz) - (double)s.off[2]) * (double)g.h[2];
            r2 = fma(dz, dz, r2);
            z = min(max(s.anc[2] + lo[2] + zz, 0), nn[2] - 1);
        }
        const double rem = smax2 - r2;
        if (!(rem > 0.0)) continue;
        const int y = min(max(s.anc[1] + lo[1] + yy, 0), nn[1] - 1);
        const float *rowp = g.J + ((long)z * g.ny + y) * g.nx;
        // the row's points inside the ball, with a rounding margin
        const float ex = fmaf(sqrtf((float)rem) * g.inv_h[0], 1.0001f, 1e-3f);
        // counted from the first, so that the ends of a centre beyond the integers (a seed may be anywhere, infinite
        // too), which the conversions hold at the largest integer, end the walk as well
        const unsigned xa = (unsigned)(int)ceilf(s.off[0] - ex);
        const int last = (int)((unsigned)(int)floorf(s.off[0] + ex) - xa);
        for (int k = q % SHARE; k <= last; k += 4 * SHARE) {
            int x[4];
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                x[u] = (int)(xa + (unsigned)(k + u * SHARE));
                v[u] = rowp[min(max((int)((unsigned)s.anc[0] + (unsigned)x[u]), 0), nn[0] - 1)];
            }
            double r[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double d = ((double)x[u] - ox) * hx;
                double d2 = fma(dy, dy, fma(d, d, 1e-290));   // never 0
                if constexpr (DIM == 3) d2 = fma(dz, dz, d2);
                const double y0 = __builtin_amdgcn_rsq(d2), g0 = d2 * y0, h0 = 0.5 * y0, e0 = fma(-h0, g0, 0.5);
                const double g1 = fma(g0, e0, g0), h1 = fma(h0, e0, h0);
                r[u] = fma(fma(-g1, g1, d2), h1, g1);
            }
            // a point outside the ball does not count, whatever its value
            if (disjoint) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double in = fma(r[u] - ain, is, in0), out = fma(r[u] - R_d, os, 0.5);
                    const double w = fmin(fmax(in, -1.0), fmin(out, 1.0));
                    acc = r[u] < smax_d ? fma(w, (double)v[u], acc) : acc;
                }
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double in = fma(r[u] - ain, is, in0), out = fma(r[u] - R_d, os, 0.5);
                    const double w = r[u] < core ? -1.0 : (r[u] < ramp ? in : (r[u] < shell ? 1.0 : out));
                    acc = r[u] < smax_d ? fma(w, (double)v[u], acc) : acc;
                }
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((t & 63) == 0) part[t >> 6] = acc;
    __syncthreads();
    if (t == 0) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < EV_T / 64; ++w) tot += part[w];
        const double meas = (double)g.h[0] * g.h[1] * (DIM == 3 ? g.h[2] : 1.0f);
        double norm = 1.0;
        for (int i = 0; i < DIM; ++i) norm *= 2.0 * (double)R;
        const double e = tot * meas / norm;
        *e_out = e;
        if (finalize) {
            DevContour o = s;
            o.e_vox = (float)e;
            if ((o.status & 0x0f) == SNK_ACTIVE) o.status = (uint8_t)((o.status & SNK_CLAMPED) | SNK_MAXITER);
            *slot = o;
        }
    }
}

enum : int { DEC_NONE = 0, DEC_UNDECIDED = 1, DEC_ACCEPT = 2, DEC_REJECT = 3 };

template <int DIM>
__device__ __forceinline__ bool overlaps(const DevContour &x, const DevContour &y, const float h[3]) {
    constexpr float RHO = DIM == 3 ? 0.79370052598409973738f : 0.70710678118654752440f;
    float d2 = 0.0f;
#pragma unroll
    for (int i = 0; i < DIM; ++i) {
        const float d = ((float)(x.anc[i] - y.anc[i]) + (x.off[i] - y.off[i])) * h[i];
        d2 = fmaf(d, d, d2);
    }
    const float thr = RHO * fmaxf(x.R, y.R);
    return sqrtf(d2) < thr;
}

// Energy that ranks contour i: E_vox for the final selection (mode 0), the last Monte-Carlo
// energy for a culling pass during evolution (mode 1) and for the final selection of star-shaped
// contours (mode 2).
__device__ __forceinline__ double rank_energy(const JobDev &a, int i, const DevContour &s) {
    return a.mode == 0 ? a.e_vox[i] : (double)s.e_mc;
}

// Whether contour i is a candidate of the selection (final: stopped contours at or below E0; culling
// pass: live contours below its threshold, or all of them during the run's grace period, for which the host
// passes a grace above every count, else 0).
__device__ __forceinline__ bool is_candidate(const JobDev &a, const DevContour &s, double e) {
    const int st = s.status & 0x0f;
    return a.mode != 1 ? (st == SNK_CONVERGED || st == SNK_MAXITER) && isfinite(e) && e <= (double)a.e0
                       : (st == SNK_ACTIVE || st == SNK_CONVERGED) && isfinite(e) &&
                             (s.iters < a.grace || e <= (double)a.e_cull);
}

template <int DIM>
__device__ __forceinline__ int grid_cell(const JobDev &a, const DevContour &s) {
    int gi[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const float pk = ((float)s.anc[k] + s.off[k]) * a.p.g.h[k];
        gi[k] = min(max((int)floorf(pk / a.cell), 0), a.G[k] - 1);
    }
    return (gi[2] * a.G[1] + gi[1]) * a.G[0] + gi[0];
}

// Outcome of the decisions for contour i: keep flag (final selection) or retirement (culling pass);
// returns 1 when it counts (kept, or retired).
__device__ __forceinline__ int apply_one(const JobDev &a, int i, int d) {
    if (a.mode != 1) {
        const uint8_t k = d == DEC_ACCEPT ? 1 : 0;
        a.st[i].keep = k;
        return k;
    }
    // culling pass: live contours that lost or are no candidates stop
    const uint8_t s8 = a.st[i].status;
    const int st = s8 & 0x0f;
    if ((st == SNK_ACTIVE || st == SNK_CONVERGED) && d != DEC_ACCEPT) {
        a.st[i].status = (uint8_t)((s8 & SNK_CLAMPED) | SNK_CULLED);
        return 1;
    }
    return 0;
}

// ---------------------------------------------------------------------------------------------
// Selection of one volume
// ---------------------------------------------------------------------------------------------
//
// Bound by latency: a few thousand contours are a few hundred waves, and each step waits for the one before.
// So the steps are few and wide: (1) clear the cells' chain heads; (2) link every candidate into its cell's
// chain, at the end of the kernel that finishes it (exact energy, or the end of evolution); (3) a group
// of lanes per candidate, one per neighbouring cell, walks the chains and lists the overlapping candidates
// with a smaller key: none, as for most, accepts at once, the others join the work list; (4) rounds over the
// work list, which read only the listed candidates' decisions; (5) the outcome. With up to kOneGroup
// contours one workgroup does (4) and (5). Finalize, before -> now (the exact energy of 55 us in the first,
// none in the second, 715 in the third): 2,000 contours 147 -> 71 us, 600 star contours 59 -> 17, 62,500 lattice
// contours 808 -> 754 (one workgroup, above 1,024 contours 14 launches, sorted the cells and re-walked them
// every round); 9,000 contours with hundreds of overlaps each 2.5 -> 0.49 ms.
constexpr int SG_T = 256;
// Contours whose outcome one workgroup writes: 8 per thread; a launch more costs about as much as 8 more.
constexpr int kOneGroup = 8192;
// A candidate's list: its length, then up to 7 indices (two 16-byte loads); a longer one walks its cells again.
constexpr int kSelList = 8;
// Contours above which grid-wide rounds come before the one-workgroup rounds: 32 candidates a step, one
// workgroup takes a thousand in the time of a few launches.
constexpr int kSelRounds = 1024;
// Batch: items that have a list (the others walk their cells again), and contours that a job's workgroup takes at
// a time.
constexpr int kListItems = 1 << 20;
constexpr int kSelChunk = 4096;

__global__ __launch_bounds__(SG_T) void sel_clear_kernel(JobDev a, int G) {
    const int i = blockIdx.x * SG_T + threadIdx.x;
    if (i < G) a.cell_start[i] = 0;
    if (i < 4) a.kept[i] = 0;   // kept, work-list length and the rounds' counters (launch_select)
}

// Links contour i (its final state s, ranking energy e) into its cell's chain if it competes.
template <int DIM>
__device__ __forceinline__ void link_one(const JobDev &a, int i, const DevContour &s, double e) {
    const bool cand = is_candidate(a, s, e);
    a.dec[i] = cand ? DEC_UNDECIDED : DEC_NONE;
    if (cand) {
        const int cell = grid_cell<DIM>(a, s);
        a.cell_of[i] = cell;
        a.items[i] = atomicExch(&a.cell_start[cell], i + 1);   // chain heads hold index + 1
    }
}

template <int DIM>
constexpr int sel_lanes() {
    return DIM == 3 ? 32 : 16;   // at least 3^DIM
}

// Lanes per candidate walk the cells around it in step. Each overlapping candidate with a smaller key is
// handed to visit(j, hit) by every lane of the group together (hit false where a lane has none); the walk
// ends when visit returns true.
template <int DIM, typename F>
__device__ __forceinline__ void walk_smaller(const JobDev &a, int i, int sub, F visit) {
    const DevContour si = a.st[i];
    const double ei = rank_energy(a, i, si);
    const int cell = a.cell_of[i];
    int next = 0;
    if (sub < (DIM == 3 ? 27 : 9)) {
        const int cx = cell % a.G[0] + sub % 3 - 1, cy = (cell / a.G[0]) % a.G[1] + sub / 3 % 3 - 1,
                  cz = DIM == 3 ? cell / (a.G[0] * a.G[1]) + sub / 9 - 1 : 0;
        if (cx >= 0 && cy >= 0 && cz >= 0 && cx < a.G[0] && cy < a.G[1] && cz < a.G[2])
            next = a.cell_start[(cz * a.G[1] + cy) * a.G[0] + cx];
    }
    constexpr int LN = sel_lanes<DIM>();
    const int lane = threadIdx.x & 63;
    const uint64_t group = ((1ull << LN) - 1) << (lane & ~(LN - 1));
    while ((__builtin_amdgcn_ballot_w64(next != 0) & group) != 0) {
        const int j = next - 1;
        bool hit = false;
        if (next != 0) {
            next = a.items[j];
            if (j != i) {
                const DevContour sj = a.st[j];
                if (overlaps<DIM>(si, sj, a.p.g.h)) {
                    const double ej = rank_energy(a, j, sj);
                    hit = ej < ei || (ej == ei && sj.id < si.id);
                }
            }
        }
        if (visit(j, hit, group)) break;
    }
}

// Step 3 for candidate i by a group of lanes: accepted at once if no overlapping candidate has a smaller key, else
// their number and the first of them into mine (null: none are kept), and true.
template <int DIM>
__device__ __forceinline__ bool list_one(const JobDev &a, int i, int sub, int *mine) {
    int total = 0;
    const int lane = threadIdx.x & 63;
    walk_smaller<DIM>(a, i, sub, [&](int j, bool hit, uint64_t group) {
        const uint64_t h = __builtin_amdgcn_ballot_w64(hit) & group;
        const int pos = total + __builtin_popcountll(h & ((1ull << lane) - 1ull));
        if (mine && hit && pos + 1 < kSelList) mine[1 + pos] = j;
        total += __builtin_popcountll(h);
        return false;
    });
    if (sub == 0) {
        if (total == 0) a.dec[i] = DEC_ACCEPT;   // no other lane reads this decision in this launch
        else if (mine) mine[0] = total;
    }
    return total != 0;
}

template <int DIM>
__global__ __launch_bounds__(SG_T) void sel_list_kernel(JobDev a, int *list, int *work, int *m) {
    constexpr int LN = sel_lanes<DIM>();
    const int i = (int)(((long)blockIdx.x * SG_T + threadIdx.x) / LN), sub = threadIdx.x & (LN - 1);
    if (i >= a.n || a.dec[i] != DEC_UNDECIDED) return;   // whole groups
    if (list_one<DIM>(a, i, sub, list + (long)i * kSelList) && sub == 0) work[atomicAdd(m, 1)] = i;
}

// A decision that other waves may be taking: a value read early only delays the reader's own decision.
template <int SCOPE>
__device__ __forceinline__ int decision(const JobDev &a, int i) {
    return __hip_atomic_load(a.dec + i, __ATOMIC_RELAXED, SCOPE);
}

// One decision step of candidate i by a group of lanes (every decision taken is final and correct whatever
// the others do meanwhile): accepted neighbour -> reject; none undecided -> accept. Returns whether it
// stays undecided. mine: its list (null: none). SCOPE: of the waves that decide concurrently.
template <int DIM, int SCOPE>
__device__ __forceinline__ bool decide_group(const JobDev &a, const int *mine, int i, int sub) {
    const int cnt = mine ? mine[0] : kSelList;
    bool accepted = false, open = false;
    if (cnt < kSelList) {
        const int d = sub < cnt ? decision<SCOPE>(a, mine[1 + sub]) : (int)DEC_REJECT;
        const uint64_t group = ((1ull << sel_lanes<DIM>()) - 1) << ((threadIdx.x & 63) & ~(sel_lanes<DIM>() - 1));
        accepted = (__builtin_amdgcn_ballot_w64(d == DEC_ACCEPT) & group) != 0;
        open = (__builtin_amdgcn_ballot_w64(d == DEC_UNDECIDED) & group) != 0;
    } else {
        walk_smaller<DIM>(a, i, sub, [&](int j, bool hit, uint64_t group) {
            const int d = hit ? decision<SCOPE>(a, j) : (int)DEC_REJECT;
            accepted = accepted || (__builtin_amdgcn_ballot_w64(d == DEC_ACCEPT) & group) != 0;
            open = open || (__builtin_amdgcn_ballot_w64(d == DEC_UNDECIDED) & group) != 0;
            return accepted;
        });
    }
    if (sub == 0 && (accepted || !open))
        __hip_atomic_store(a.dec + i, accepted ? (int)DEC_REJECT : (int)DEC_ACCEPT, __ATOMIC_RELAXED, SCOPE);
    return !accepted && open;
}

// Step 4, grid-wide. Round r: skipped when round r - 1 left nothing undecided; counts what it leaves
// undecided in left[r % 3] and clears left[(r + 1) % 3] for the next round.
template <int DIM>
__global__ __launch_bounds__(SG_T) void sel_round_kernel(JobDev a, const int *list, const int *work, const int *m, int r,
                                                         int *left) {
    if (r > 0 && *(volatile int *)&left[(r + 2) % 3] == 0) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) left[(r + 1) % 3] = 0;
    constexpr int LN = sel_lanes<DIM>();
    const int k = (int)(((long)blockIdx.x * SG_T + threadIdx.x) / LN), sub = threadIdx.x & (LN - 1);
    if (k >= *m) return;   // whole groups
    const int i = work[k];
    if (__shfl(decision<__HIP_MEMORY_SCOPE_AGENT>(a, i), 0, LN) != DEC_UNDECIDED) return;
    if (decide_group<DIM, __HIP_MEMORY_SCOPE_AGENT>(a, list + (long)i * kSelList, i, sub) && sub == 0) atomicAdd(&left[r % 3], 1);
}

// Steps 4 and 5 by one workgroup: rounds until nothing on the work list is undecided, then (apply) the outcome
// of every contour.
template <int DIM>
__global__ __launch_bounds__(SEL_T) void sel_finish_kernel(JobDev a, const int *list, const int *work, const int *mp,
                                                           int apply) {
    constexpr int LN = sel_lanes<DIM>();
    const int t = threadIdx.x, sub = t & (LN - 1);
    const int m = *mp;
    constexpr int SCOPE = __HIP_MEMORY_SCOPE_WORKGROUP;
    bool any = m > 0;
    while (any) {
        int local = 0;
        for (int k = t / LN; k < m; k += SEL_T / LN) {
            const int i = work[k];
            if (__shfl(decision<SCOPE>(a, i), 0, LN) == DEC_UNDECIDED)
                local |= decide_group<DIM, SCOPE>(a, list + (long)i * kSelList, i, sub) ? 1 : 0;
        }
        __threadfence_block();
        any = __syncthreads_or(local) != 0;
    }
    if (!apply) return;
    int count = 0;
    for (int i = t; i < a.n; i += SEL_T) count += apply_one(a, i, decision<SCOPE>(a, i));
    for (int o = 32; o > 0; o >>= 1) count += __shfl_xor(count, o, 64);
    if ((t & 63) == 0 && count) atomicAdd(a.kept, (unsigned long long)count);
}

// The outcome of every decision, grid-wide (after the decisions are complete).
__global__ __launch_bounds__(SG_T) void sel_apply_kernel(JobDev a) {
    const int i = blockIdx.x * SG_T + threadIdx.x;
    const int c = i < a.n ? apply_one(a, i, a.dec[i]) : 0;
    const int total = __syncthreads_count(c);
    if (threadIdx.x == 0 && total) atomicAdd(a.kept, (unsigned long long)total);
}

// Step 2 where no exact energy is formed: contours still ACTIVE become MAXITER (mode 2), candidates are linked.
template <int DIM>
__global__ __launch_bounds__(SG_T) void sel_link_kernel(JobDev a) {
    const int i = blockIdx.x * SG_T + threadIdx.x;
    if (i >= a.n) return;
    DevContour s = a.st[i];
    if (a.mode == 2 && (s.status & 0x0f) == SNK_ACTIVE) {
        s.status = (uint8_t)((s.status & SNK_CLAMPED) | SNK_MAXITER);
        a.st[i].status = s.status;
    }
    link_one<DIM>(a, i, s, rank_energy(a, i, s));
}

// A culling pass without competition judges each contour alone.
__global__ __launch_bounds__(SG_T) void cull_alone_kernel(JobDev a) {
    const int i = blockIdx.x * SG_T + threadIdx.x;
    int c = 0;
    if (i < a.n) {
        const DevContour s = a.st[i];
        c = apply_one(a, i, is_candidate(a, s, (double)s.e_mc) ? DEC_ACCEPT : DEC_NONE);
    }
    const int total = __syncthreads_count(c);
    if (threadIdx.x == 0 && total) atomicAdd(a.kept, (unsigned long long)total);
}

template <int DIM>
__global__ __launch_bounds__(ev_threads<DIM>()) void energy_link_kernel(JobDev a) {
    const int cid = blockIdx.x;
    energy_one<DIM>(a.p, a.st + cid, a.e_vox + cid, true);
    if (threadIdx.x == 0) {
        // this thread wrote the state and energy it reads here
        const DevContour s = a.st[cid];
        link_one<DIM>(a, cid, s, a.e_vox[cid]);
    }
}

template <int DIM>
hipError_t select_plain(const JobDev &j, int *list, int *work, hipStream_t s) {
    const int G = j.G[0] * j.G[1] * j.G[2];
    const int bn = (j.n + SG_T - 1) / SG_T;
    // kept counter, then three more 64-bit words: work-list length and the rounds' three counters
    int *m = reinterpret_cast<int *>(j.kept + 1);
    int *left = m + 1;
    const bool alone = j.mode == 1 && !j.compete;
    hipLaunchKernelGGL(sel_clear_kernel, dim3(alone ? 1 : (std::max(G, 4) + SG_T - 1) / SG_T), dim3(SG_T), 0, s, j,
                       alone ? 0 : G);
    if (alone) {
        hipLaunchKernelGGL(cull_alone_kernel, dim3(bn), dim3(SG_T), 0, s, j);
        return hipGetLastError();
    }
    if (j.mode == 0)
        hipLaunchKernelGGL(energy_link_kernel<DIM>, dim3(j.n), dim3(ev_threads<DIM>()), 0, s, j);
    else
        hipLaunchKernelGGL(sel_link_kernel<DIM>, dim3(bn), dim3(SG_T), 0, s, j);
    constexpr int per = SG_T / sel_lanes<DIM>();
    const int bg = (j.n + per - 1) / per;
    hipLaunchKernelGGL(sel_list_kernel<DIM>, dim3(bg), dim3(SG_T), 0, s, j, list, work, m);
    const int rounds = j.n > kOneGroup ? 6 : (j.n > kSelRounds ? 2 : 0);
    for (int r = 0; r < rounds; ++r)
        hipLaunchKernelGGL(sel_round_kernel<DIM>, dim3(bg), dim3(SG_T), 0, s, j, list, work, m, r, left);
    const bool apply = j.n <= kOneGroup;
    hipLaunchKernelGGL(sel_finish_kernel<DIM>, dim3(1), dim3(SEL_T), 0, s, j, list, work, m, apply ? 1 : 0);
    if (!apply) hipLaunchKernelGGL(sel_apply_kernel, dim3(bn), dim3(SG_T), 0, s, j);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Selection of a batch
// ---------------------------------------------------------------------------------------------
//
// The same steps over the items of many jobs: clear, link at the end of the exact energy, list, and a workgroup per
// job for the rounds and the outcome, which takes kSelChunk contours at a time and gathers their undecided
// candidates in LDS. Bound by latency, 4 to 5 us a launch: 24 jobs of up to 300 contours 14 us, against 60 for one
// workgroup per job that sorted its cells and walked them again every round.

__global__ __launch_bounds__(SEL_T) void sel_clear_batch_kernel(const JobDev *jobs, const int2 *job_list) {
    const JobDev &j = jobs[__builtin_amdgcn_readfirstlane(job_list[blockIdx.x].x)];
    const int G = j.G[0] * j.G[1] * j.G[2];
    for (int c = threadIdx.x; c < G; c += SEL_T) j.cell_start[c] = 0;
}

template <int DIM>
__global__ __launch_bounds__(ev_threads<DIM>()) void energy_link_batch_kernel(const JobDev *jobs, const int2 *items) {
    const int2 it = items[blockIdx.x];
    const int job = __builtin_amdgcn_readfirstlane(it.x), cid = __builtin_amdgcn_readfirstlane(it.y);
    const JobDev &j = jobs[job];
    energy_one<DIM>(j.p, j.st + cid, j.e_vox + cid, true);
    if (threadIdx.x == 0) {
        // this thread wrote the state and energy it reads here
        const DevContour s = j.st[cid];
        link_one<DIM>(j, cid, s, j.e_vox[cid]);
    }
}

template <int DIM>
__global__ __launch_bounds__(SG_T) void sel_list_batch_kernel(const JobDev *jobs, const int2 *items, int n_items,
                                                              int *list) {
    constexpr int LN = sel_lanes<DIM>();
    const long q = ((long)blockIdx.x * SG_T + threadIdx.x) / LN;
    if (q >= n_items) return;   // whole groups
    const int2 it = items[q];
    const JobDev a = jobs[it.x];
    if (a.dec[it.y] != DEC_UNDECIDED) return;
    list_one<DIM>(a, it.y, threadIdx.x & (LN - 1), q < kListItems ? list + q * kSelList : nullptr);
}

// job_list: the job's row of the table and its first item (its contours' items follow each other).
template <int DIM>
__global__ __launch_bounds__(SEL_T) void sel_finish_batch_kernel(const JobDev *jobs, const int2 *job_list,
                                                                 const int *list) {
    __shared__ int open[kSelChunk];
    __shared__ int m;
    constexpr int LN = sel_lanes<DIM>();
    constexpr int SCOPE = __HIP_MEMORY_SCOPE_WORKGROUP;
    const int t = threadIdx.x, sub = t & (LN - 1);
    const int base = __builtin_amdgcn_readfirstlane(job_list[blockIdx.x].y);
    const JobDev &a = jobs[__builtin_amdgcn_readfirstlane(job_list[blockIdx.x].x)];
    const int n = a.n;
    bool any = n > 0;
    while (any) {
        int local = 0;
        for (int c0 = 0; c0 < n; c0 += kSelChunk) {
            if (t == 0) m = 0;
            __syncthreads();
            for (int i = c0 + t; i < min(n, c0 + kSelChunk); i += SEL_T)
                if (decision<SCOPE>(a, i) == DEC_UNDECIDED) open[atomicAdd(&m, 1)] = i;
            __syncthreads();
            const int cnt = m;
            for (int k = t / LN; k < cnt; k += SEL_T / LN) {
                const int i = open[k];
                const long q = (long)base + i;
                local |= decide_group<DIM, SCOPE>(a, q < kListItems ? list + q * kSelList : nullptr, i, sub) ? 1 : 0;
            }
            __threadfence_block();
            __syncthreads();
        }
        any = __syncthreads_or(local) != 0;
    }
    int count = 0;
    for (int i = t; i < n; i += SEL_T) count += apply_one(a, i, decision<SCOPE>(a, i));
    for (int o = 32; o > 0; o >>= 1) count += __shfl_xor(count, o, 64);
    if ((t & 63) == 0 && count) atomicAdd(a.kept, (unsigned long long)count);
}

template <int DIM>
hipError_t select_batch(const JobDev *jobs, const int2 *items, int n_items, const int2 *job_list, int n_jobs, int *list,
                        hipStream_t s) {
    hipLaunchKernelGGL(sel_clear_batch_kernel, dim3(n_jobs), dim3(SEL_T), 0, s, jobs, job_list);
    if (n_items > 0) {
        constexpr int per = SG_T / sel_lanes<DIM>();
        hipLaunchKernelGGL(energy_link_batch_kernel<DIM>, dim3(n_items), dim3(ev_threads<DIM>()), 0, s, jobs, items);
        hipLaunchKernelGGL(sel_list_batch_kernel<DIM>, dim3((n_items + per - 1) / per), dim3(SG_T), 0, s, jobs, items,
                           n_items, list);
        hipLaunchKernelGGL(sel_finish_batch_kernel<DIM>, dim3(n_jobs), dim3(SEL_T), 0, s, jobs, job_list, list);
    }
    return hipGetLastError();
}

}  // namespace

namespace {
__global__ __launch_bounds__(256) void compact_active_kernel(const DevContour *st, int n, int *idx, int *count) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const bool act = i < n && (st[i].status & 0x0f) == SNK_ACTIVE;
    // one atomic per wave: the active lanes take consecutive slots in lane order
    const unsigned long long m = __builtin_amdgcn_ballot_w64(act);
    const int lane = threadIdx.x & 63;
    int base = 0;
    if (lane == 0 && m) base = atomicAdd(count, __popcll(m));
    base = __shfl(base, 0, 64);
    if (act) idx[base + __popcll(m & ((1ull << lane) - 1ull))] = i;
}
}  // namespace

hipError_t launch_compact_active(const DevContour *st, int n, int *idx, int *count, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(compact_active_kernel, dim3((n + 255) / 256), dim3(256), 0, s, st, n, idx, count);
    return hipGetLastError();
}

hipError_t launch_select(const JobDev &j, int dim, int *list, int *work, hipStream_t s) {
    if (j.n <= 0) return hipSuccess;
    return dim == 2 ? select_plain<2>(j, list, work, s) : select_plain<3>(j, list, work, s);
}

size_t select_list_ints(int64_t n) { return (size_t)n * kSelList; }

hipError_t launch_select_batch(const JobDev *jobs, const int2 *items, int n_items, const int2 *job_list, int n_jobs,
                               int *list, int dim, hipStream_t s) {
    if (n_jobs <= 0) return hipSuccess;
    return dim == 2 ? select_batch<2>(jobs, items, n_items, job_list, n_jobs, list, s)
                    : select_batch<3>(jobs, items, n_items, job_list, n_jobs, list, s);
}

size_t select_batch_ints(size_t n_items) { return std::min(n_items, (size_t)kListItems) * kSelList; }

}  // namespace snk
