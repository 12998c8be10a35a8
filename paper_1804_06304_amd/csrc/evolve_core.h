// Evolution kernel: gradient descent of independent snakuscules with Monte-Carlo sums.
//
// A group of G lanes owns one contour and runs its iterations back to back; contours are
// independent during evolution (Sec. II-D), so there is no grid-wide synchronisation. G is 16 or 32
// (several contours share one wave64), 64 (one wave per contour) or 128/256 (a workgroup of 2/4
// waves per contour). Per iteration n the group
//   1. reads, for each antithetic pair m, the ray direction u = Q(n) T[k] already divided by the
//      voxel spacing, and the radial jitter xi. These are state-independent: the Philox4x32-10 draws
//      (rotation Q(n) at counter (0, n, id, 0), Shoemake's uniform quaternion in 3D or an angle in
//      2D; table row k = floor(x0 D / 2^32) and xi from counter (m, n, id, 1)) are produced for a
//      block of K iterations at once by all lanes of the group, one draw per lane, and the
//      rotations are applied in the following iteration, so each costs about 1/K of a draw per lane
//      and iteration;
//   2. walks pair-points (m, l): both rays +u and -u at the common radius
//      s = s_max ((l + xi)/L)^(1/d), s_max = R + dR/2 (uniform in the ball, Sec. II-E), issuing the
//      trilinear (bilinear) gathers of both points before consuming them. The two points share the
//      radius, hence S and its ramp memberships;
//   3. evaluates the four-region weight S (Sec. II-B, Eq. (5)) and accumulates
//      A = sum S I, B_R = sum dS/dR I and B_c = -sum dS/dr I u (per pair: the ramp coefficient times
//      I(+u) + I(-u) for A and B_R, times I(+u) - I(-u) for B_c; B_c is kept in voxel units);
//   4. reduces the sums in a fixed order (DPP row shifts/rotations inside a wave, then per-wave
//      partials in wave order through LDS), so every lane of the group holds identical totals;
//   5. applies the descent step of Eqs. (7)-(15) in (c, R) form: E = A/(2R)^d,
//      dE/dR = (B_R - (d/R) A)/(2R)^d, dE/dc = B_c/(2R)^d, eps = eps0/sqrt(n),
//      dR = -(eps/2) dE/dR, dc = -(eps/2) dE/dc (the p,q steps of Eqs. (12)-(15) mapped through
//      c = (p+q)/2, R = (q_x - p_x)/2), clamps R, re-anchors c, and tests OUT / convergence.
// Sub-wave groups (run_group) hold the state in every lane; whole-wave groups (run_wave) step the axes of
// the centre in lanes of their own.
//
// Volume layouts: plain FP32 [z][y][x] (2^d/2 eight-byte pair loads per point), or "quad": one
// 16-byte record per voxel holding J(x,y), J(x+1,y), J(x,y+1), J(x+1,y+1) of its plane (one 16-byte
// load per point in 2D, two in 3D). Both hold exact copies of the smoothed volume.
//
// Two launches share the per-contour routine: one group per contour of a single volume, and a
// batched launch over a device table of (job, contour) items (one workgroup per item, optionally
// persistent with a work queue).
#pragma once

#include <math.h>

#include "snk_internal.h"

namespace snk {

namespace {

constexpr uint32_t kBufferWord3 = 0x00020000u;  // raw buffer descriptor, gfx9 family

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// The rounds stay a loop of two rounds: fully unrolled, the compiler keeps all twenty round keys in scalar
// registers for the whole kernel and spills other uniform values to make room; one round per step costs
// two register moves a round (the words change places).
__device__ __forceinline__ void philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                         uint32_t k1, uint32_t out[4]) {
#pragma unroll 1
    for (int r = 0; r < 5; ++r) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // one 32 x 32 -> 64-bit product gives both halves
            const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
            const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
            const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
            const uint32_t n0 = hi1 ^ c1 ^ k0;
            const uint32_t n2 = hi0 ^ c3 ^ k1;
            c0 = n0;
            c1 = lo1;
            c2 = n2;
            c3 = lo0;
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
    }
    out[0] = c0;
    out[1] = c1;
    out[2] = c2;
    out[3] = c3;
}

// (2*(x >> 9) + 1) * 2^-24: exact in FP32, strictly inside (0, 1).
__device__ __forceinline__ float unit_open(uint32_t x) {
    return (float)((x >> 9) * 2u + 1u) * 5.9604644775390625e-08f;
}

// Rotation Q (row-major, acting on column vectors) from the Philox words of counter (0, n, id, 0).
// Evaluated operation by operation (no multiply-add contraction), so every kernel instance and build
// rounds it alike.
template <int DIM>
__device__ __forceinline__ void rotation_from(const uint32_t x[4], float Q[9]) {
#pragma clang fp contract(off)
    if constexpr (DIM == 2) {
        float s, c;
        sincospif(2.0f * unit_open(x[0]), &s, &c);
        Q[0] = c;
        Q[1] = -s;
        Q[2] = 0.0f;
        Q[3] = s;
        Q[4] = c;
        Q[5] = 0.0f;
        Q[6] = 0.0f;
        Q[7] = 0.0f;
        Q[8] = 1.0f;
    } else {
        const float u1 = unit_open(x[0]), u2 = unit_open(x[1]), u3 = unit_open(x[2]);
        const float a = sqrtf(1.0f - u1), b = sqrtf(u1);
        float s1, c1, s2, c2;
        sincospif(2.0f * u2, &s1, &c1);
        sincospif(2.0f * u3, &s2, &c2);
        const float qx = a * s1, qy = a * c1, qz = b * s2, qw = b * c2;
        Q[0] = 1.0f - 2.0f * (qy * qy + qz * qz);
        Q[1] = 2.0f * (qx * qy - qw * qz);
        Q[2] = 2.0f * (qx * qz + qw * qy);
        Q[3] = 2.0f * (qx * qy + qw * qz);
        Q[4] = 1.0f - 2.0f * (qx * qx + qz * qz);
        Q[5] = 2.0f * (qy * qz - qw * qx);
        Q[6] = 2.0f * (qx * qz - qw * qy);
        Q[7] = 2.0f * (qy * qz + qw * qx);
        Q[8] = 1.0f - 2.0f * (qx * qx + qy * qy);
    }
}

// ---------------------------------------------------------------------------------------------
// Group shape and LDS layout
// ---------------------------------------------------------------------------------------------

template <int G>
struct Grp {
    static constexpr int NT = G < 64 ? 64 : G;       // threads per workgroup
    static constexpr int CPB = G < 64 ? 64 / G : 1;  // contours per workgroup
    static constexpr int WAVES = NT / 64;
};

// Iterations per block of draws. A block takes ceil(K (MH + 1) / G) rounds of one draw per lane;
// K is the smallest block size (at least two: the rotation of a block is applied one iteration
// after its draws) whose rounds per iteration come within 30% of the ideal (MH + 1) / G, else the
// one with the fewest rounds per iteration.
__host__ __device__ __forceinline__ int block_iters(int G, int MH) {
    const int per = MH + 1;
    int best = 2;
    float best_cost = 1e30f;
    for (int K = 2; K <= 16; ++K) {
        const float cost = (float)((K * per + G - 1) / G) / (float)K;
        if (cost * (float)G <= 1.3f * (float)per) return K;
        if (cost < best_cost) {
            best_cost = cost;
            best = K;
        }
    }
    return best;
}

// Floats of one contour's draw buffers (two blocks), a multiple of 4.
__host__ __device__ __forceinline__ int draw_floats(int G, int MH) {
    const int K = block_iters(G, MH);
    return 2 * K * (4 * MH + 12);
}

// One contour's draw buffers: for each of 2 blocks x K iterations,
//   pu[m] = (u_x/h_x, u_y/h_y, u_z/h_z, xi) per pair m (between the two phases pu[m].x holds the
//   table row k), rot = Q (9 floats, 12 reserved).
struct Draws {
    float4 *pu;
    float *rot;
    int K, MH;
    __device__ __forceinline__ Draws(float *base, int G, int MH_) {
        MH = MH_;
        K = block_iters(G, MH_);
        pu = reinterpret_cast<float4 *>(base);
        rot = base + 2 * K * 4 * MH;
    }
    __device__ __forceinline__ int slot(int buf, int s) const { return buf * K + s; }
};

// j -> (j / d, j % d) for small j, without an integer division.
__device__ __forceinline__ void divmod_small(int j, int d, float inv_d, int &q, int &r) {
    q = (int)(((float)j + 0.5f) * inv_d);
    r = j - q * d;
    if (r < 0) {
        q -= 1;
        r += d;
    } else if (r >= d) {
        q += 1;
        r -= d;
    }
}

// Phase 1 of block b: the Philox draws of its K iterations (n_first .. n_first + K - 1), one per
// lane: pair draws -> table row k (parked in pu.x) and xi; rotation draws -> Q (ROT = false: none, for
// directions that stay fixed).
template <int DIM, int G, bool ROT = true>
__device__ __forceinline__ void draws_phase1(const Draws &d, int buf, uint32_t n_first, uint32_t id,
                                             const JobParams &p, int gl) {
    const int per = d.MH + 1;
    const int total = d.K * per;
    const float inv = 1.0f / (float)per;
    for (int j = gl; j < total; j += G) {
        int s, r;
        divmod_small(j, per, inv, s, r);
        const bool pair = r < d.MH;
        uint32_t x[4];
        philox10(pair ? (uint32_t)r : 0u, n_first + (uint32_t)s, id, pair ? 1u : 0u, p.key0, p.key1, x);
        const int sl = d.slot(buf, s);
        if (pair) {
            d.pu[sl * d.MH + r].x = __int_as_float((int)__umulhi(x[0], (uint32_t)p.D));
            d.pu[sl * d.MH + r].w = unit_open(x[1]);
        } else if constexpr (ROT) {
            float Q[9];
            if (p.flags & 1) {
#pragma unroll
                for (int i = 0; i < 9; ++i) Q[i] = (i % 4 == 0) ? 1.0f : 0.0f;
            } else {
                rotation_from<DIM>(x, Q);
            }
#pragma unroll
            for (int i = 0; i < 9; ++i) d.rot[sl * 12 + i] = Q[i];
        }
    }
}

// Phase 2 of block b (one iteration after phase 1): u = Q T[k] / h for every pair of the block.
template <int DIM, int G>
__device__ __forceinline__ void draws_phase2(const Draws &d, int buf, const JobParams &p, int gl) {
    const int total = d.K * d.MH;
    const float inv = 1.0f / (float)d.MH;
    for (int j = gl; j < total; j += G) {
        int s, m;
        divmod_small(j, d.MH, inv, s, m);
        const int sl = d.slot(buf, s);
        float4 &o = d.pu[sl * d.MH + m];
        const int k = __float_as_int(o.x);
        const float *Q = d.rot + sl * 12;
        float t[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < DIM; ++i) t[i] = p.dirs[k * DIM + i];
        float u[3];
#pragma unroll
        for (int i = 0; i < DIM; ++i) {
            float acc = 0.0f;
#pragma unroll
            for (int jj = 0; jj < DIM; ++jj) acc = fmaf(Q[i * 3 + jj], t[jj], acc);
            u[i] = acc * p.g.inv_h[i];
        }
        o.x = u[0];
        o.y = u[1];
        o.z = DIM == 3 ? u[2] : 0.0f;
    }
}

// A record in constant memory (the kernel's arguments, or a table no kernel of the launch writes) read where
// it is needed: the compiler would load every field before the loop and, out of scalar registers, spill them
// to lanes of a vector register; through a pointer it cannot see through, a field is one scalar load at
// its use. For what an iteration seldom needs.
template <typename T>
using Cold = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ Cold<T> cold(Cold<T> p) {
    asm volatile("" : "+s"(p));
    return p;
}

// Draw buffers of a whole-wave group: pairs pu[m] = (u_x/h_x, u_y/h_y, u_z/h_z, xi) of two blocks of K
// iterations (the one in use and the next), and the rotations of KR iterations (a multiple of K).
//   - Pairs: 64 draws are one wave's pass. A block's passes go to the group's waves in turn, starting with
//     another wave each block, so a block of one pass (K MH <= 64) costs each wave a pass every WAVES
//     blocks. The host picks K (draw_plan) so that the passes are nearly full.
//   - Rotations: one lane draws an iteration's, so a pass gives KR of them; apart from the pairs' passes
//     because a pass that holds even one rotation runs its whole code (about 150 instructions in 3D),
//     which with both in the same pass was a third of the draws' cost.
// Schedule within iteration it = b K + sl: at sl = 0 each wave's first pass of block b + 1 draws and fetches
// its table rows after the iteration's gathers (whose registers are free then) and applies the rotation
// at its end, so the fetch's latency hides behind the reduction and the step; at the end of sl = K - 1 a
// wave draws the next KR rotations when block b + 2 is their first. Both ends lie behind the iteration's
// reduction barrier, so with K >= 2 every value is written at least one barrier before another wave reads
// it, and after the last read of what it overwrites.
template <int DIM>
constexpr int rot_floats() {
    return DIM == 3 ? 9 : 2;
}

template <int DIM, int G>
struct WaveDraws {
    static constexpr int WAVES = G / 64;
    float4 *pu;
    float *rot;
    int K, KR, MH, T, passes;
    float inv_mh;
    __device__ __forceinline__ WaveDraws(float *base, int K_, int KR_, int MH_) {
        K = K_;
        KR = KR_;
        MH = MH_;
        T = K * MH;
        passes = (T + 63) >> 6;
        inv_mh = 1.0f / (float)MH;
        pu = reinterpret_cast<float4 *>(base);
        rot = base + 8 * T;
    }
    // rotations of iterations n_first .. n_first + KR - 1, one per lane of the calling wave
    __device__ __forceinline__ void rotations(uint32_t n_first, uint32_t id, Cold<JobParams> cp, int lane) const {
        const Cold<JobParams> p = cold(cp);
        for (int s = lane; s < KR; s += 64) {
            float Q[9] = {1.0f, 0.0f, 0.0f, 0.0f, 1.0f, 0.0f, 0.0f, 0.0f, 1.0f};
            if (!(p->flags & 1)) {
                uint32_t x[4];
                philox10(0u, n_first + (uint32_t)s, id, 0u, p->key0, p->key1, x);
                rotation_from<DIM>(x, Q);
            }
            float *o = rot + s * rot_floats<DIM>();
            if constexpr (DIM == 3) {
#pragma unroll
                for (int i = 0; i < 9; ++i) o[i] = Q[i];
            } else {
                o[0] = Q[0];   // cos
                o[1] = Q[3];   // sin
            }
        }
    }
    // one pair's draw: its place, table row (not yet rotated) and jitter
    struct Pending {
        float t[3], xi;
        int s, m;
        bool on;
    };
    __device__ __forceinline__ Pending begin(int r, uint32_t n_first, uint32_t id, Cold<JobParams> cp, int lane) const {
        const Cold<JobParams> p = cold(cp);
        Pending d;
        const int j = r * 64 + lane;
        d.on = j < T;
        divmod_small(d.on ? j : 0, MH, inv_mh, d.s, d.m);
        uint32_t x[4];
        philox10((uint32_t)d.m, n_first + (uint32_t)d.s, id, 1u, p->key0, p->key1, x);
        const int k = (int)__umulhi(x[0], (uint32_t)p->D);
        d.xi = unit_open(x[1]);
        d.t[0] = d.t[1] = d.t[2] = 0.0f;
#pragma unroll
        for (int i = 0; i < DIM; ++i) d.t[i] = p->dirs[k * DIM + i];
        return d;
    }
    // u = Q t / h of the block's iteration s, whose rotation is entry rot0 + s
    __device__ __forceinline__ void finish(const Pending &d, int buf, int rot0, Cold<JobParams> cp) const {
        if (!d.on) return;
        const Cold<JobParams> p = cold(cp);
        const float *q = rot + (rot0 + d.s) * rot_floats<DIM>();
        float Q[9];
        if constexpr (DIM == 3) {
#pragma unroll
            for (int i = 0; i < 9; ++i) Q[i] = q[i];
        } else {
            Q[0] = q[0];
            Q[1] = -q[1];
            Q[3] = q[1];
            Q[4] = q[0];
        }
        float u[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < DIM; ++i) {
            float acc = 0.0f;
#pragma unroll
            for (int jj = 0; jj < DIM; ++jj) acc = fmaf(Q[i * 3 + jj], d.t[jj], acc);
            u[i] = acc * p->g.inv_h[i];
        }
        pu[(buf * K + d.s) * MH + d.m] = make_float4(u[0], u[1], u[2], d.xi);
    }
};

// ---------------------------------------------------------------------------------------------
// Reductions (fixed order; every lane of a group ends with identical totals)
// ---------------------------------------------------------------------------------------------

template <int CTRL, int ROWS = 0xf, bool BC = true>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, BC));
}

// Butterfly over the 16 lanes of a DPP row (rotations are symmetric, so all lanes agree bitwise).
__device__ __forceinline__ float row_sum16(float v) {
    v += dpp<0x128>(v);  // row_ror:8
    v += dpp<0x124>(v);  // row_ror:4
    v += dpp<0x122>(v);  // row_ror:2
    v += dpp<0x121>(v);  // row_ror:1
    return v;
}

// Sum of the wave in lane 63 (row shifts, then row broadcasts).
__device__ __forceinline__ float wave_sum_to_63(float v) {
    v += dpp<0x111>(v);             // row_shr:1
    v += dpp<0x112>(v);             // row_shr:2
    v += dpp<0x114>(v);             // row_shr:4
    v += dpp<0x118>(v);             // row_shr:8
    v += dpp<0x142, 0xa, false>(v); // row_bcast:15
    v += dpp<0x143, 0xc, false>(v); // row_bcast:31
    return v;
}

// Maximum of the wave in lane 63 (row shifts, then row broadcasts; values are >= 0 here, so the
// zero filled in by the shifts is harmless).
__device__ __forceinline__ float wave_max_to_63(float v) {
    v = fmaxf(v, dpp<0x111>(v));             // row_shr:1
    v = fmaxf(v, dpp<0x112>(v));             // row_shr:2
    v = fmaxf(v, dpp<0x114>(v));             // row_shr:4
    v = fmaxf(v, dpp<0x118>(v));             // row_shr:8
    v = fmaxf(v, dpp<0x142, 0xa, false>(v)); // row_bcast:15
    v = fmaxf(v, dpp<0x143, 0xc, false>(v)); // row_bcast:31
    return v;
}

// Adds a value's copies in the two halves of the wave (lane i and lane i ^ 32), then in the two rows
// of each half (lane i and lane i ^ 16); both partners add the same two operands in the same order.
__device__ __forceinline__ float cross_row_sum(float x) {
    auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = __uint_as_float(h[0]) + __uint_as_float(h[1]);   // x[i mod 32] + x[32 + i mod 32]
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);            // even row + odd row of the half
}

// Totals over the 64 lanes of a wave of NR = 4 or 5 per-lane values. Values 0..3 are reduced together:
// lanes exchange values so that after two quad steps each lane holds the quad's sum of one value,
// j = 2 (lane & 1) + ((lane >> 1) & 1); the row and cross-row steps then add the copies of that value
// (the same value sits in lanes i, i + 4, i + 8, ...). A fifth value takes the same steps on its own.
// Every value is added over the same tree whatever its place, and the order of every addition is fixed,
// so the totals do not depend on timing. On return x holds, in lane i, the total of value 0, 2, 1, 3 for
// i & 3 = 0, 1, 2, 3, and z in every lane that of value 4.
template <int NR>
__device__ __forceinline__ void wave_quads(const float *v, float &x, float &z) {
    static_assert(NR == 4 || NR == 5, "four or five sums");
    const bool b0 = __builtin_amdgcn_inverse_ballot_w64(0xAAAAAAAAAAAAAAAAull);
    const bool b1 = __builtin_amdgcn_inverse_ballot_w64(0xCCCCCCCCCCCCCCCCull);
    // lane pairs (2i, 2i + 1): the even lane keeps values 0 and 1, the odd one 2 and 3
    const float k0 = b0 ? v[2] : v[0], k1 = b0 ? v[3] : v[1];
    const float s0 = b0 ? v[0] : v[2], s1 = b0 ? v[1] : v[3];
    const float w0 = k0 + dpp<0xB1>(s0);   // quad_perm [1, 0, 3, 2]
    const float w1 = k1 + dpp<0xB1>(s1);
    // lanes i and i ^ 2: keep w_b1, add the partner's copy of the same value
    const float keep = b1 ? w1 : w0, send = b1 ? w0 : w1;
    x = keep + dpp<0x4E>(send);           // quad_perm [2, 3, 0, 1]
    z = 0.0f;
    if constexpr (NR == 5) {
        z = v[4] + dpp<0xB1>(v[4]);
        z = z + dpp<0x4E>(z);
    }
    x += dpp<0x128>(x);                   // row_ror:8
    x += dpp<0x124>(x);                   // row_ror:4
    if constexpr (NR == 5) {
        z += dpp<0x128>(z);
        z += dpp<0x124>(z);
    }
    x = cross_row_sum(x);
    if constexpr (NR == 5) z = cross_row_sum(z);
}

// Sum over a sub-wave group of 16 or 32 lanes.
template <int G>
__device__ __forceinline__ float group_sum(float v) {
    v = row_sum16(v);
    if constexpr (G == 32)
        v += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));  // lane ^ 16
    return v;
}

// Sum over a wave, in every lane.
__device__ __forceinline__ float wave_sum(float v) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_sum_to_63(v)), 63));
}

// ---------------------------------------------------------------------------------------------
// Volume access
// ---------------------------------------------------------------------------------------------

struct __attribute__((packed, aligned(4))) Pair {
    float lo, hi;
};

// The 2^d corner values of one trilinear (bilinear) sample, in the order
// v000 v100 v010 v110 v001 v101 v011 v111.
template <int DIM>
struct Corners {
    float v[DIM == 3 ? 8 : 4];
};

template <int DIM, int LAYOUT>
struct Vol {
    static constexpr bool kSmall = LAYOUT != kGlobalPlain;  // 24-bit index arithmetic
    const float *J;
    __amdgpu_buffer_rsrc_t rsrc;
    int nx, nxy;
    int so1, so2, so3;  // byte offsets of the neighbour loads (buffer layouts)
    __device__ __forceinline__ Vol(const Geometry &g) {
        nx = g.nx;
        nxy = g.nx * g.ny;
        J = g.J;
        so1 = so2 = so3 = 0;
        if constexpr (LAYOUT == kBufferPlain) {
            so1 = nx * 4;
            so2 = nxy * 4;
            so3 = (nxy + nx) * 4;
            rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)g.J, (short)0, (int)((long)nxy * g.nz * 4),
                                                     (int)kBufferWord3);
        } else if constexpr (LAYOUT == kBufferQuad) {
            so2 = nxy * 16;
            rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)g.Jq, (short)0, (int)((long)nxy * g.nz * 16),
                                                     (int)kBufferWord3);
        } else if constexpr (LAYOUT == kBufferPair) {
            so2 = nxy * 8;
            rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)g.Jq, (short)0, (int)((long)nxy * (DIM == 3 ? g.nz : 1) * 8),
                                                     (int)kBufferWord3);
        }
    }
    // One voxel value (plain layouts).
    __device__ __forceinline__ float load1(long idx) const {
        if constexpr (LAYOUT == kBufferPlain) {
            return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)idx * 4, 0, 0));
        } else if constexpr (LAYOUT == kBufferPair) {
            return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)idx * 8, 0, 0));
        } else {
            return J[idx];
        }
    }
    // Loads the corners of the cell whose lower corner has linear voxel index base + rel (< 2^31 for
    // the buffer layouts; base uniform, so its byte offset stays in a scalar register).
    __device__ __forceinline__ void load(long rel, long base, Corners<DIM> &c) const {
        if constexpr (LAYOUT == kBufferQuad) {
            const int vo = (int)rel * 16 + (int)base * 16;
            const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, 0, 0);
            c.v[0] = __uint_as_float(a.x);
            c.v[1] = __uint_as_float(a.y);
            c.v[2] = __uint_as_float(a.z);
            c.v[3] = __uint_as_float(a.w);
            if constexpr (DIM == 3) {
                const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, so2, 0);
                c.v[4] = __uint_as_float(b.x);
                c.v[5] = __uint_as_float(b.y);
                c.v[6] = __uint_as_float(b.z);
                c.v[7] = __uint_as_float(b.w);
            }
        } else if constexpr (LAYOUT == kBufferPair) {
            // (J(x,y), J(x,y+1)) then (J(x+1,y), J(x+1,y+1)), of plane z and then of plane z+1
            const int vo = (int)rel * 8 + (int)base * 8;
            const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, 0, 0);
            c.v[0] = __uint_as_float(a.x);
            c.v[2] = __uint_as_float(a.y);
            c.v[1] = __uint_as_float(a.z);
            c.v[3] = __uint_as_float(a.w);
            if constexpr (DIM == 3) {
                const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, so2, 0);
                c.v[4] = __uint_as_float(b.x);
                c.v[6] = __uint_as_float(b.y);
                c.v[5] = __uint_as_float(b.z);
                c.v[7] = __uint_as_float(b.w);
            }
        } else if constexpr (LAYOUT == kBufferPlain) {
            const int vo = (int)rel * 4 + (int)base * 4;
            const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(rsrc, vo, 0, 0);
            const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(rsrc, vo, so1, 0);
            c.v[0] = __uint_as_float(a.x);
            c.v[1] = __uint_as_float(a.y);
            c.v[2] = __uint_as_float(b.x);
            c.v[3] = __uint_as_float(b.y);
            if constexpr (DIM == 3) {
                const u32x2 e = __builtin_amdgcn_raw_buffer_load_b64(rsrc, vo, so2, 0);
                const u32x2 f = __builtin_amdgcn_raw_buffer_load_b64(rsrc, vo, so3, 0);
                c.v[4] = __uint_as_float(e.x);
                c.v[5] = __uint_as_float(e.y);
                c.v[6] = __uint_as_float(f.x);
                c.v[7] = __uint_as_float(f.y);
            }
        } else {
            const float *q = J + (base + rel);
            const Pair a = *reinterpret_cast<const Pair *>(q);
            const Pair b = *reinterpret_cast<const Pair *>(q + nx);
            c.v[0] = a.lo;
            c.v[1] = a.hi;
            c.v[2] = b.lo;
            c.v[3] = b.hi;
            if constexpr (DIM == 3) {
                const Pair e = *reinterpret_cast<const Pair *>(q + nxy);
                const Pair f = *reinterpret_cast<const Pair *>(q + (long)nxy + nx);
                c.v[4] = e.lo;
                c.v[5] = e.hi;
                c.v[6] = f.lo;
                c.v[7] = f.hi;
            }
        }
    }
};

// Corner reads from a box of the smoothed volume staged in LDS (x fastest; nx = box row length,
// nxy = box plane size). Indices are relative to the box, so they stay small.
template <int DIM>
struct TileVol {
    static constexpr bool kSmall = true;
    const float *t;
    int nx, nxy;
    __device__ __forceinline__ void load(long rel, long base, Corners<DIM> &c) const {
        const float *q = t + ((int)base + (int)rel);
        c.v[0] = q[0];
        c.v[1] = q[1];
        c.v[2] = q[nx];
        c.v[3] = q[nx + 1];
        if constexpr (DIM == 3) {
            const float *r = q + nxy;
            c.v[4] = r[0];
            c.v[5] = r[1];
            c.v[6] = r[nx];
            c.v[7] = r[nx + 1];
        }
    }
};

template <int DIM>
__device__ __forceinline__ float trilerp(const Corners<DIM> &c, const float f[3]) {
    const float a0 = fmaf(f[0], c.v[1] - c.v[0], c.v[0]);
    const float a1 = fmaf(f[0], c.v[3] - c.v[2], c.v[2]);
    const float b0 = fmaf(f[1], a1 - a0, a0);
    if constexpr (DIM == 2) {
        return b0;
    } else {
        const float a2 = fmaf(f[0], c.v[5] - c.v[4], c.v[4]);
        const float a3 = fmaf(f[0], c.v[7] - c.v[6], c.v[6]);
        const float b1 = fmaf(f[1], a3 - a2, a2);
        return fmaf(f[2], b1 - b0, b0);
    }
}

// Trilinear (bilinear) value with the same operations as trilerp, and its gradient with respect to
// the voxel coordinates in the same cell.
template <int DIM>
__device__ __forceinline__ float trilerp_grad(const Corners<DIM> &c, const float f[3], float g[3]) {
    const float d0 = c.v[1] - c.v[0], d1 = c.v[3] - c.v[2];
    const float a0 = fmaf(f[0], d0, c.v[0]);
    const float a1 = fmaf(f[0], d1, c.v[2]);
    const float e0 = a1 - a0;
    const float b0 = fmaf(f[1], e0, a0);
    const float q0 = fmaf(f[1], d1 - d0, d0);
    if constexpr (DIM == 2) {
        g[0] = q0;
        g[1] = e0;
        g[2] = 0.0f;
        return b0;
    } else {
        const float d2 = c.v[5] - c.v[4], d3 = c.v[7] - c.v[6];
        const float a2 = fmaf(f[0], d2, c.v[4]);
        const float a3 = fmaf(f[0], d3, c.v[6]);
        const float e1 = a3 - a2;
        const float b1 = fmaf(f[1], e1, a2);
        const float q1 = fmaf(f[1], d3 - d2, d2);
        const float gz = b1 - b0;
        g[0] = fmaf(f[2], q1 - q0, q0);
        g[1] = fmaf(f[2], e1 - e0, e0);
        g[2] = gz;
        return fmaf(f[2], gz, b0);
    }
}

// Per-contour quantities of one iteration that the sampler reads.
template <int DIM>
struct Frame {
    int anc[3];
    float off[3];
    long base;     // linear index of the anchor voxel
    float smax;
    // weight S(r; R) (Sec. II-B): inner core -1 up to rho R - dr/2, ramp of width dr = rho dR, shell
    // +1 up to R - dR/2, outer ramp of width dR down to 0 at R + dR/2; half-open intervals
    float ain, R;          // centres of the inner and outer ramps
    float hd, hD;          // half widths dr/2 and dR/2
    float is, os;          // ramp slopes 2/dr and 1/dR
    float rho_is;          // rho * is
};

// floor(x) as an integer in one instruction (|x| far below 2^31 here).
__device__ __forceinline__ int floor_to_int(float x) {
    int i;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(x));
    return i;
}

// Point x = anchor + off + rad * du (voxel units) -> corner index, relative to the anchor voxel
// (CLAMP: to voxel 0), and fractions. CLAMP = false is used only when every sample of the iteration is
// known to lie inside, where both agree. SMALL: the row and plane strides fit 24-bit multiplies
// (buffer layouts).
// out (CLAMP only, may be null): per axis 0.0 where the coordinate lies beyond the volume's faces
// (the clamped interpolant is flat there), else 1.0; the last face itself counts as inside.
template <int DIM, bool CLAMP, bool SMALL>
__device__ __forceinline__ long locate(const Frame<DIM> &fr, const int *n, int nx, int nxy, const float w[3],
                                       float f[3], float *in = nullptr) {
    if constexpr (!CLAMP) {
        int i[3] = {0, 0, 0};
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            i[a] = floor_to_int(w[a]);
            f[a] = __builtin_amdgcn_fractf(w[a]);
        }
        if constexpr (SMALL) {
            int rel = __mul24(i[1], nx) + i[0];
            if constexpr (DIM == 3) rel += __mul24(i[2], nxy);
            return rel;
        } else {
            long rel = (long)i[1] * nx + i[0];
            if constexpr (DIM == 3) rel += (long)i[2] * nxy;
            return rel;
        }
    } else {
        long idx = 0;
        const long stride[3] = {1, nx, nxy};
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            const float fl = floorf(w[a]);
            int i = fr.anc[a] + (int)fl;
            float fa = w[a] - fl;
            if (in) in[a] = (i < 0 || i > n[a] - 1 || (i == n[a] - 1 && fa > 0.0f)) ? 0.0f : 1.0f;
            if (i < 0) {
                i = 0;
                fa = 0.0f;
            } else if (i > n[a] - 2) {
                i = n[a] - 2;
                fa = 1.0f;
            }
            f[a] = fa;
            idx += (long)i * stride[a];
        }
        return idx;
    }
}

template <int DIM>
__device__ __forceinline__ float cube_or_square_root(float tau) {
    if constexpr (DIM == 3) {
        // tau in (0, 1), never denormal: 2^(log2(tau)/3) on the transcendental unit
        return __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(tau) * 0.333333343267f);
    } else {
        return __builtin_amdgcn_sqrtf(tau);
    }
}

// Sums of one lane for one iteration over pair-points q = gl, gl + G, ... < P (pair m = q / L,
// radial index l = q % L), U pair-points in flight.
// FULL: L = 16 and G U divides P, so every pass of every lane holds U valid pair-points, all at the lane's
// radial index gl % 16 (pairs gl / 16 + k G / 16), and the passes are uniform: no per-pair-point index
// stepping or validity tests. The arithmetic of each pair-point is the same in both forms.
// n: the volume's size (CLAMP only). GRADI: the centre sums are sum S grad I (voxel-coordinate gradient of the interpolant, zero along
// axes beyond a face) instead of sum -dS/dr I u / h.
template <int DIM, int G, int U, bool CLAMP, bool GRADI = false, bool FULL = false, typename V>
__device__ __forceinline__ void lane_sums(const V &vol, const int *n, const Frame<DIM> &fr, const float4 *pu,
                                          int P, int L, float invL, int gl, int l0, int m0, int dl, int dm,
                                          float acc[2 + DIM]) {
    int l = l0, m = FULL ? gl >> 4 : m0;
    const float lf = (float)(gl & 15);
    if constexpr (FULL) invL = 0.0625f;
    for (int q = FULL ? 0 : gl; q < P; q += G * U) {
        Corners<DIM> cp[U], cm[U];
        float fp[U][3], fm[U][3], d1s[U], d2s[U];
        float inp[U][3], inm[U][3];
        int mk[U];
        bool ok[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if constexpr (FULL) {
                ok[k] = true;
                mk[k] = m + k * (G / 16);
            } else {
                ok[k] = q + k * G < P;
                mk[k] = ok[k] ? m : 0;
            }
            const float4 d = pu[mk[k]];
            const float tau = ((FULL ? lf : (float)l) + d.w) * invL;
            const float e = cube_or_square_root<DIM>(tau);
            const float rad = fr.smax * e;
            // offsets from the ramp centres, fused explicitly so every instance rounds them alike
            d1s[k] = fmaf(fr.smax, e, -fr.ain);
            d2s[k] = fmaf(fr.smax, e, -fr.R);
            float wp[3] = {0.0f, 0.0f, 0.0f}, wm[3] = {0.0f, 0.0f, 0.0f};
            const float du[3] = {d.x, d.y, d.z};
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                wp[a] = fmaf(rad, du[a], fr.off[a]);
                wm[a] = fmaf(-rad, du[a], fr.off[a]);
            }
            constexpr bool SMALL = V::kSmall;
            const long ip = locate<DIM, CLAMP, SMALL>(fr, n, vol.nx, vol.nxy, wp, fp[k],
                                                      GRADI && CLAMP ? inp[k] : nullptr);
            const long im = locate<DIM, CLAMP, SMALL>(fr, n, vol.nx, vol.nxy, wm, fm[k],
                                                      GRADI && CLAMP ? inm[k] : nullptr);
            vol.load(ip, CLAMP ? 0 : fr.base, cp[k]);
            vol.load(im, CLAMP ? 0 : fr.base, cm[k]);
            if constexpr (!FULL) {
                l += dl;
                m += dm;
                if (l >= L) {
                    l -= L;
                    m += 1;
                }
            }
        }
        if constexpr (FULL) m += U * (G / 16);
        // branch-free: a pair-point past P (it read pair 0, in bounds) gets zero weights, so its
        // gathers are consumed unconditionally and those of all U pair-points stay in flight
        // together
#pragma unroll
        for (int k = 0; k < U; ++k) {
            float gp[3], gm[3];
            const float Ip = GRADI ? trilerp_grad<DIM>(cp[k], fp[k], gp) : trilerp<DIM>(cp[k], fp[k]);
            const float Im = GRADI ? trilerp_grad<DIM>(cm[k], fm[k], gm) : trilerp<DIM>(cm[k], fm[k]);
            const float d1 = d1s[k], d2 = d2s[k];
            const bool r1 = d1 >= -fr.hd && d1 < fr.hd;   // inner ramp
            const bool r2 = d2 >= -fr.hD && d2 < fr.hD;   // outer ramp
            const float sin_ = __builtin_amdgcn_fmed3f(d1 * fr.is, -1.0f, 1.0f);
            const float sout = __builtin_amdgcn_fmed3f(fmaf(-d2, fr.os, 0.5f), 0.0f, 1.0f);
            // the inner profile is +1 wherever the outer one is below 1 (R >= the geometric
            // minimum keeps the regions disjoint), and vice versa
            const float S = ok[k] ? fminf(sin_, sout) : 0.0f;
            const float cC = ok[k] ? (r1 ? fr.is : (r2 ? -fr.os : 0.0f)) : 0.0f;  // dS/dr on the ramps
            const float cR = ok[k] ? (r1 ? -fr.rho_is : -cC) : 0.0f;               // dS/dR on the ramps
            const float Is = Ip + Im, Id = Ip - Im;
            acc[0] = fmaf(S, Is, acc[0]);
            acc[1] = fmaf(cR, Is, acc[1]);
            if constexpr (GRADI) {
                // both points share the radius, hence S
#pragma unroll
                for (int a = 0; a < DIM; ++a) {
                    const float gsum = CLAMP ? fmaf(gp[a], inp[k][a], gm[a] * inm[k][a]) : gp[a] + gm[a];
                    acc[2 + a] = fmaf(S, gsum, acc[2 + a]);
                }
            } else {
                const float g = cC * Id;
                const float4 d = pu[mk[k]];
                acc[2] = fmaf(-g, d.x, acc[2]);
                acc[3] = fmaf(-g, d.y, acc[3]);
                if constexpr (DIM == 3) acc[4] = fmaf(-g, d.z, acc[4]);
            }
        }
    }
}

// Exact sums of one lane (flags bit 1): the lattice points of the box around the ball of radius
// s_max, those inside the ball counted (the point set of Eq. (5)), I = J at the voxel itself
// (clamp-to-edge outside the volume when CLAMP). Box points q = gl, gl + G, ..., x fastest; P
// points are evaluated per pass with their loads issued first. Bound by issue, some 60 instructions per
// point, 13 points per lane and iteration: so a lane's place in the box takes no integer division and no loop (600
// contours, 60 iterations, 256 lanes: 343 -> 305 us; seven points per pass 330).
template <int DIM, int G, bool CLAMP, int LAYOUT>
__device__ __forceinline__ void lattice_sums(const Vol<DIM, LAYOUT> &vol, const int *n, const Frame<DIM> &fr, const float hh[3],
                                             const float inv_h[3], int gl, float acc[2 + DIM]) {
    constexpr int P = 4;
    int lo[3] = {0, 0, 0}, cnt[3] = {1, 1, 1};
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        const float e = fr.smax * inv_h[a];
        lo[a] = (int)ceilf(fr.off[a] - e);
        cnt[a] = (int)floorf(fr.off[a] + e) - lo[a] + 1;
    }
    const int total = cnt[0] * cnt[1] * cnt[2];
    // the lane's first point and the step of G points as digits of the box (a step carries at most once per digit)
    const float i0 = 1.0f / (float)cnt[0], i1 = 1.0f / (float)cnt[1];
    int x, y, z, sx, sy, sz;
    divmod_small(gl, cnt[0], i0, y, x);
    divmod_small(y, cnt[1], i1, z, y);
    divmod_small(G, cnt[0], i0, sy, sx);
    divmod_small(sy, cnt[1], i1, sz, sy);
    const float smax2 = fr.smax * fr.smax;
    for (int q0 = gl; q0 < total; q0 += G * P) {
        float I[P], d[P][3], r2[P];
        bool in[P];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int j[3] = {lo[0] + x, lo[1] + y, lo[2] + z};
            x += sx;
            y += sy;
            z += sz;
            if (x >= cnt[0]) {
                x -= cnt[0];
                y += 1;
            }
            if (y >= cnt[1]) {
                y -= cnt[1];
                z += 1;
            }
            r2[k] = 0.0f;
            d[k][0] = d[k][1] = d[k][2] = 0.0f;
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                d[k][a] = ((float)j[a] - fr.off[a]) * hh[a];
                r2[k] = fmaf(d[k][a], d[k][a], r2[k]);
            }
            in[k] = q0 + k * G < total && r2[k] < smax2;
            long idx;
            if constexpr (CLAMP) {
                idx = 0;
                const long stride[3] = {1, vol.nx, vol.nxy};
#pragma unroll
                for (int a = 0; a < DIM; ++a) idx += (long)min(max(fr.anc[a] + j[a], 0), n[a] - 1) * stride[a];
            } else if constexpr (LAYOUT != kGlobalPlain) {
                int rel = __mul24(j[1], vol.nx) + j[0];
                if constexpr (DIM == 3) rel += __mul24(j[2], vol.nxy);
                idx = fr.base + rel;
            } else {
                long rel = (long)j[1] * vol.nx + j[0];
                if constexpr (DIM == 3) rel += (long)j[2] * vol.nxy;
                idx = fr.base + rel;
            }
            I[k] = in[k] ? vol.load1(idx) : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (!in[k]) continue;
            const float r = __builtin_amdgcn_sqrtf(r2[k]);
            const float inv_r = r > 0.0f ? __builtin_amdgcn_rcpf(r) : 0.0f;
            const float d1 = r - fr.ain, d2 = r - fr.R;
            const bool r1 = d1 >= -fr.hd && d1 < fr.hd;   // inner ramp
            const bool ro = d2 >= -fr.hD && d2 < fr.hD;   // outer ramp
            const float sin_ = __builtin_amdgcn_fmed3f(d1 * fr.is, -1.0f, 1.0f);
            const float sout = __builtin_amdgcn_fmed3f(fmaf(-d2, fr.os, 0.5f), 0.0f, 1.0f);
            const float S = fminf(sin_, sout);
            const float cC = r1 ? fr.is : (ro ? -fr.os : 0.0f);
            const float cR = r1 ? -fr.rho_is : -cC;
            acc[0] = fmaf(S, I[k], acc[0]);
            acc[1] = fmaf(cR, I[k], acc[1]);
            const float g = cC * I[k] * inv_r;   // dS/dr I / r; u = d / r
#pragma unroll
            for (int a = 0; a < DIM; ++a) acc[2 + a] = fmaf(-g, d[k][a] * inv_h[a], acc[2 + a]);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// LDS tile of the sample ball
// ---------------------------------------------------------------------------------------------

// A box of the smoothed volume held in LDS by one whole-wave group: voxels lo[a] .. lo[a] + n[a] - 1
// per axis, x fastest (n[2] = 1 in 2D). An iteration whose samples, trilinear corners included,
// all fall inside the box reads its corners from LDS; the box is staged again only when the ball
// leaves it. It is staged with a margin, so a contour that moves and grows slowly keeps its box
// for many iterations, and its corners stop costing scattered global loads.
struct Tile {
    int lo[3], n[3];
    bool valid;
};

constexpr int kTileMargin = 2;  // voxels added on each side of the ball's range, when they fit

// Voxel range lo .. hi per axis that the corners of an iteration's samples can touch (the ball of
// radius s_max around the centre, with the same rounding margin as the interior test).
template <int DIM>
__device__ __forceinline__ void ball_range(const Frame<DIM> &fr, const float inv_h[3], int lo[3], int hi[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = hi[a] = 0;
        if (a < DIM) {
            const float e = fmaf(fr.smax * inv_h[a], 1.0001f, 1e-3f);
            lo[a] = fr.anc[a] + (int)floorf(fr.off[a] - e);
            hi[a] = fr.anc[a] + (int)floorf(fr.off[a] + e) + 1;
        }
    }
}

// New box for the range lo .. hi (inside the volume): the largest margin of kTileMargin .. 0
// voxels per side whose box holds at most `cap` voxels, clamped to the volume. False if even the
// bare range does not fit.
template <int DIM>
__device__ __forceinline__ bool choose_tile(const int lo[3], const int hi[3], const int nvol[3], int cap, Tile &t) {
    for (int m = kTileMargin; m >= 0; --m) {
        int n[3] = {1, 1, 1};
        int size = 1;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            n[a] = min(hi[a] - lo[a] + 1 + 2 * m, nvol[a]);
            size *= n[a];
        }
        if (size <= cap) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                t.n[a] = n[a];
                t.lo[a] = a < DIM ? min(max(lo[a] - m, 0), nvol[a] - n[a]) : 0;
            }
            t.valid = true;
            return true;
        }
    }
    t.valid = false;
    return false;
}

// All G lanes copy the box from the plain FP32 volume into LDS, 8 loads in flight per lane. The
// caller synchronises the group before the box is read.
template <int G>
__device__ __forceinline__ void stage_tile(float *tile, const float *J, int nx, int nxy, const Tile &t, int gl) {
    const int n0 = t.n[0], n1 = t.n[1];
    const int total = n0 * n1 * t.n[2];
    const float *src = J + ((long)t.lo[2] * nxy + (long)t.lo[1] * nx + t.lo[0]);
    // element e = gl + k G of the box -> (x, y, z), advanced by G without a division
    int x = gl % n0, y = (gl / n0) % n1, z = gl / (n0 * n1);
    const int sx = G % n0, sy = G / n0;
    constexpr int B = 8;
    for (int e0 = gl; e0 < total; e0 += B * G) {
        float v[B];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            v[k] = e0 + k * G < total ? src[(long)z * nxy + y * nx + x] : 0.0f;
            x += sx;
            if (x >= n0) {
                x -= n0;
                y += 1;
            }
            y += sy;
            while (y >= n1) {
                y -= n1;
                z += 1;
            }
        }
#pragma unroll
        for (int k = 0; k < B; ++k)
            if (e0 + k * G < total) tile[e0 + k * G] = v[k];
    }
}

// ---------------------------------------------------------------------------------------------
// Per-contour iteration loop
// ---------------------------------------------------------------------------------------------

// Copy of a record that every lane reads at the same address, forced into scalar registers (the
// table lives in memory the kernel also writes, so the compiler would otherwise keep it per lane).
template <typename T>
__device__ __forceinline__ T uniform_copy(const T *src) {
    static_assert(sizeof(T) % 4 == 0, "word-sized record");
    T out;
    const uint32_t *in = reinterpret_cast<const uint32_t *>(src);
    uint32_t *o = reinterpret_cast<uint32_t *>(&out);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) o[i] = __builtin_amdgcn_readfirstlane(in[i]);
    return out;
}

// A value identical in every lane of a whole-wave group, moved to a scalar register (frees vector
// registers; sub-wave groups keep per-lane values).
template <int G>
__device__ __forceinline__ float uni(float v) {
    if constexpr (G >= 64) return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
    else return v;
}
template <int G>
__device__ __forceinline__ int uni(int v) {
    if constexpr (G >= 64) return __builtin_amdgcn_readfirstlane(v);
    else return v;
}

// A value that the compiler cannot see through: what is formed from the lane's number would otherwise be
// formed before the loop and kept in a register of its own for all of it.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Soft repulsion of one contour: its neighbour list holds cnt (ascending) of the contours in a->snap; -1: off.
struct Repel {
    Cold<EvolveArgs> a;
    int cid, cnt;
};

// Per-iteration quantities of the weight for radius R.
template <int DIM, int G>
__device__ __forceinline__ void set_frame(Frame<DIM> &fr, const JobParams &p, float smax, float ain, float R) {
    constexpr float RHO = DIM == 3 ? 0.79370052598409973738f : 0.70710678118654752440f;
    fr.smax = smax;
    fr.ain = ain;
    fr.R = R;
    fr.hd = uni<G>(0.5f * RHO * p.dR);
    fr.hD = uni<G>(0.5f * p.dR);
    fr.is = p.in_slope;
    fr.os = p.out_slope;
    fr.rho_is = uni<G>(RHO * p.in_slope);
}

// Sub-wave groups (G = 16 or 32, several contours per wave64): run up to n_iter iterations of the group's
// contour (slot == nullptr: no contour), stopping early when it leaves SNK_ACTIVE. All lanes of the
// workgroup call this; the loop and its barriers are workgroup-uniform. Every lane holds its contour's state.
template <int DIM, int G, int U, bool TRACE, int LAYOUT, bool EXACT = false>
__device__ void run_group(const JobParams &p, DevContour *slot, int n_iter, float *trace_row, float *lds_draws,
                          unsigned long long *counter) {
    static_assert(G < 64, "whole waves: run_wave");
    constexpr int NR = 2 + DIM;
    constexpr float RHO = DIM == 3 ? 0.79370052598409973738f : 0.70710678118654752440f;
    constexpr float BALL = DIM == 3 ? 4.18879020478639098462f : 3.14159265358979323846f;
    const int gl = threadIdx.x & (G - 1);

    DevContour s{};
    s.status = SNK_OUT;
    if (slot) s = *slot;
    const int n0 = s.iters;
    const int budget = ((s.status & 0x0f) == SNK_ACTIVE && slot) ? min(n_iter, 0x7fffffff - n0) : 0;
    const int MH = p.M / 2;
    const int P = MH * p.L;
    const Draws dr(lds_draws, G, MH);
    const uint32_t id = s.id;
    const Vol<DIM, LAYOUT> vol(p.g);
    const int nvol[3] = {p.g.nx, p.g.ny, p.g.nz};
    const float inv_h[3] = {p.g.inv_h[0], p.g.inv_h[1], p.g.inv_h[2]};
    const float hh[3] = {p.g.h[0], p.g.h[1], p.g.h[2]};

    if (!EXACT && budget > 0) draws_phase1<DIM, G>(dr, 0, (uint32_t)(n0 + 1), id, p, gl);
    __syncthreads();
    if (!EXACT && budget > 0) draws_phase2<DIM, G>(dr, 0, p, gl);
    __syncthreads();

    // lane's first pair-point and its step
    const int L = p.L;
    const float invL = 1.0f / (float)L;
    const int l0 = gl % L, m0 = gl / L;
    const int dl = G % L, dm = G / L;

    int anc[3] = {s.anc[0], s.anc[1], s.anc[2]};
    float off[3] = {s.off[0], s.off[1], s.off[2]};
    float R = s.R;
    int n = n0;
    uint8_t status = s.status;
    int streak = s.streak;
    float e_mc = s.e_mc;
    const float inv_npts = 1.0f / (float)(p.M * p.L);
    const float tol2 = p.conv_tol * p.conv_tol;
    int ran = 0;
    int cull_next = p.cull_first;  // this launch's next culling pass point (-1: none)

    for (int it = 0;; ++it) {
        const bool active = it < budget && (status & 0x0f) == SNK_ACTIVE;
        if (__builtin_amdgcn_ballot_w64(active) == 0) break;
        float acc[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) acc[k] = 0.0f;
        Frame<DIM> fr;
        bool interior = true;
        if (active) {
            const int blk = it / dr.K, sl = it - blk * dr.K;
            if (!EXACT && sl == 0)
                draws_phase1<DIM, G>(dr, (blk + 1) & 1, (uint32_t)(n0 + 1 + (blk + 1) * dr.K), id, p, gl);
            if (!EXACT && sl == 1) draws_phase2<DIM, G>(dr, (blk + 1) & 1, p, gl);

            set_frame<DIM, G>(fr, p, R + 0.5f * p.dR, RHO * R, R);
            long base = 0;
            const long stride[3] = {1, vol.nx, vol.nxy};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                fr.anc[a] = anc[a];
                fr.off[a] = off[a];
            }
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
                base += (long)anc[a] * stride[a];
                // clamping can be skipped when the whole sample ball (with a rounding margin) is
                // interior
                const float ext = fmaf(fr.smax * inv_h[a], 1.0001f, 1e-3f);
                interior = interior && (off[a] - ext > (float)(-anc[a])) &&
                           (off[a] + ext < (float)(nvol[a] - 1 - anc[a]));
            }
            fr.base = base;
            if constexpr (EXACT) {
                if (interior)
                    lattice_sums<DIM, G, false, LAYOUT>(vol, nvol, fr, hh, inv_h, gl, acc);
                else
                    lattice_sums<DIM, G, true, LAYOUT>(vol, nvol, fr, hh, inv_h, gl, acc);
            } else {
                const float4 *pu = dr.pu + dr.slot(blk & 1, sl) * MH;
                if (interior)
                    lane_sums<DIM, G, U, false>(vol, nvol, fr, pu, P, L, invL, gl, l0, m0, dl, dm, acc);
                else
                    lane_sums<DIM, G, U, true>(vol, nvol, fr, pu, P, L, invL, gl, l0, m0, dl, dm, acc);
            }
        }

        float tot[NR];
#pragma unroll
        for (int k = 0; k < NR; ++k) tot[k] = group_sum<G>(acc[k]);

        // descent step, identical in every lane of the group
        if (active) {
            // no multiply-add contraction in the step: every instance (with or without the optional
            // terms of run_wave) rounds it operation by operation, so their results agree bit for bit
#pragma clang fp contract(off)
            n += 1;
            const float smax = fr.smax;
            float smax_d = smax;
#pragma unroll
            for (int i = 1; i < DIM; ++i) smax_d *= smax;
            // Monte-Carlo: V/N; exact: the voxel measure
            const float scale = EXACT ? hh[0] * hh[1] * (DIM == 3 ? hh[2] : 1.0f) : BALL * smax_d * inv_npts;
            const float A = scale * tot[0];
            const float BR = scale * tot[1];
            const float inv2R = __builtin_amdgcn_rcpf(2.0f * R);
            float inv_norm = inv2R;
#pragma unroll
            for (int i = 1; i < DIM; ++i) inv_norm *= inv2R;
            const float E = A * inv_norm;
            const float gR = (BR - (2.0f * DIM) * inv2R * A) * inv_norm;
            const float eps = p.eps0 * __builtin_amdgcn_rsqf((float)n);
            const float half_eps = 0.5f * eps;
            const float dRs = -half_eps * gR;
            const float kc = -half_eps * scale * inv_norm;
            float doff[3] = {0.0f, 0.0f, 0.0f}, dc[3] = {0.0f, 0.0f, 0.0f};
            float dc2 = 0.0f;
#pragma unroll
            for (int i = 0; i < DIM; ++i) {
                doff[i] = kc * tot[2 + i];   // voxel units (B_c was accumulated against u / h)
                dc[i] = doff[i] * hh[i];
            }
#pragma unroll
            for (int i = 0; i < DIM; ++i) dc2 = fmaf(dc[i], dc[i], dc2);
            if (TRACE && gl == 0) {
                float *row = trace_row;
                row[0] = A;
                row[1] = BR;
                for (int i = 0; i < 3; ++i) row[2 + i] = i < DIM ? scale * tot[2 + i] * hh[i] : 0.0f;
                row[5] = E;
                row[6] = dRs;
                for (int i = 0; i < 3; ++i) row[7 + i] = dc[i];
                row[10] = (float)n;
                row[11] = R;
                row[12] = eps;
                row[13] = row[14] = row[15] = 0.0f;
            }
            float Rn = R + dRs;
            uint8_t flag = status & SNK_CLAMPED;
            if (Rn < p.r_lo) {
                Rn = p.r_lo;
                flag = SNK_CLAMPED;
            }
            if (Rn > p.r_hi) {
                Rn = p.r_hi;
                flag = SNK_CLAMPED;
            }
            const float dRe = Rn - R;
            const bool small = dRe * dRe < tol2 && dc2 < tol2;
            R = Rn;
            e_mc = E;
            bool finite = isfinite(Rn) && isfinite(E);
#pragma unroll
            for (int i = 0; i < DIM; ++i) {
                off[i] += doff[i];
                finite = finite && isfinite(off[i]);
            }
            uint8_t st = SNK_ACTIVE;
            if (!finite) {
                st = SNK_NONFINITE;
            } else {
#pragma unroll
                for (int i = 0; i < DIM; ++i) {
                    if (fabsf(off[i]) >= 0.5f) {
                        const float k = rintf(off[i]);
                        anc[i] += (int)k;
                        off[i] -= k;
                    }
                    if (off[i] < (float)(-anc[i]) || off[i] > (float)(nvol[i] - 1 - anc[i])) st = SNK_OUT;
                }
            }
            if (st == SNK_ACTIVE) {
                streak = small ? min(streak + 1, 255) : 0;
                if (p.conv_window > 0 && streak >= p.conv_window) st = SNK_CONVERGED;
            }
            if (it == cull_next) {
                if (st == SNK_ACTIVE && !(E <= p.cull_thr)) st = SNK_CULLED;
                cull_next = cull_next + p.cull_every <= p.cull_last ? cull_next + p.cull_every : -1;
            }
            status = (uint8_t)(st | flag);
            ++ran;
        }
        __syncthreads();  // orders this iteration's LDS draws before later reads
    }

    if (slot && gl == 0 && budget > 0) {
        DevContour o = s;
        for (int i = 0; i < 3; ++i) {
            o.anc[i] = anc[i];
            o.off[i] = off[i];
        }
        o.R = R;
        o.e_mc = e_mc;
        o.iters = n;
        o.status = status;
        o.streak = (uint8_t)streak;
        *slot = o;
        atomicAdd(counter, (unsigned long long)ran);
    }
}

// Whole-wave groups (G = 64, 128 or 256 lanes, one contour per workgroup): run up to n_iter iterations of
// the contour, stopping at iteration `target` or when it leaves SNK_ACTIVE.
//
// What bounds an iteration is instruction issue: one contour's iterations are a serial chain, a wave issues
// one vector instruction per four cycles, and 4 to 8 samples per lane are few against the code around them.
// So that code is kept short:
//   - the step works on the axes in parallel: after the quad reduction lane i holds the total of A, x, y, z
//     (2D: A, x, y, B_R) for i & 3 = 0 .. 3, and the centre's offset, its bounds and the spacing live in the
//     same lanes, so the step, the interior and box tests and the OUT test each take one instruction for all
//     axes; only the three offsets the gathers need move to scalar registers;
//   - what hardly ever happens (a new anchor voxel, OUT, a value that is not finite) is one test of all of it
//     together and a branch;
//   - factors that do not depend on the sums are formed before the waves meet;
//   - FULL instances (L = 16 and whole passes) step no per-pair-point indices;
//   - the draws: see WaveDraws.
// Vector instructions per wave and iteration, before -> now, and the evolve's time: slab (3D, two waves, 512
// pair-points, boxes) 748 -> 546, 2.70 -> 2.34 ms (2.20 with the box's present size); 8192^2 image (one wave, 128
// pair-points, from pairs) 280 -> 231, 5.1 -> 4.2 ms (248 from boxes, which spare the pre-pass the pairs); 62,500
// lattice contours (four waves' work) 456 -> 323, 10.6 -> 9.1 ms, and 7.8 ms by two waves with boxes.
//
// STAGE: iterations whose ball fits a box of tile_cap voxels read their corners from an LDS box, the others
// from the volume in LAYOUT. lds: draws, the waves' partial sums, the box.
// cp: p in constant memory. PG < G (FULL): PG lanes do the work of G, wave by wave: the sums of each of
// the G / 64 waves are formed and reduced in turn, so the totals are those of G lanes bit for bit, and what an
// iteration costs beside its samples is paid by fewer waves.
template <int DIM, int G, int U, bool TRACE, int LAYOUT, bool EXACT, bool STAGE, bool GRADI, bool FULL, int PG = G>
__device__ void run_wave(const JobParams &p, Cold<JobParams> cp, DevContour *slot, int n_iter, int target,
                         float *trace_row, float *lds, int draw_k, int rot_k, unsigned long long *counter,
                         int tile_cap, const Repel rp) {
    static_assert(G >= 64, "whole waves");
    static_assert(!STAGE || !EXACT, "LDS boxes are staged by Monte-Carlo groups");
    constexpr int NR = 2 + DIM;
    constexpr int WAVES = PG / 64;    // waves of the workgroup
    constexpr int PARTS = G / 64;     // waves whose sums the totals are made of
    static_assert(PG == G || (FULL && PG < G), "fewer lanes than the group has: FULL instances");
    constexpr float RHO = DIM == 3 ? 0.79370052598409973738f : 0.70710678118654752440f;
    constexpr float BALL = DIM == 3 ? 4.18879020478639098462f : 3.14159265358979323846f;
    constexpr uint64_t AXES = DIM == 3 ? 0xE : 0x6;         // lanes 1 .. DIM: the axes
    constexpr uint64_t LAST = DIM == 3 ? 0x8 : 0x4;         // lane of the last axis
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;

    const DevContour s = uniform_copy(slot);
    const int n0 = s.iters;
    const int budget = (s.status & 0x0f) == SNK_ACTIVE ? min(n_iter, target - n0) : 0;
    if (budget <= 0) return;   // uniform over the workgroup
    const int MH = p.M / 2;
    const int P = MH * p.L;
    const int L = p.L;
    const uint32_t id = s.id;
    const Vol<DIM, LAYOUT> vol(p.g);
    const WaveDraws<DIM, PG> dr(lds, draw_k, rot_k, MH);
    float *lds_red = lds + (EXACT ? 0 : wave_draw_floats(DIM, draw_k, rot_k, MH));
    float *lds_axis = lds_red + (PARTS > 1 ? 16 * PARTS : 0);
    float *lds_tile = lds_axis + 32 * WAVES;
    const int nb = EXACT ? 1 : dr.KR / dr.K;   // blocks per set of rotations
    if constexpr (!EXACT) {
        // the last wave draws the rotations while the others' first passes draw and fetch their table rows
        typename WaveDraws<DIM, PG>::Pending pend;
        if (wave < dr.passes) pend = dr.begin(wave, (uint32_t)(n0 + 1), id, cp, lane);
        if (wave == WAVES - 1) dr.rotations((uint32_t)(n0 + 1), id, cp, lane);
        __syncthreads();
        if (wave < dr.passes) dr.finish(pend, 0, 0, cp);
        for (int r = wave + WAVES; r < dr.passes; r += WAVES)
            dr.finish(dr.begin(r, (uint32_t)(n0 + 1), id, cp, lane), 0, 0, cp);
        __syncthreads();
        if (nb == 1) {
            if (wave == WAVES - 1) dr.rotations((uint32_t)(n0 + 1 + dr.K), id, cp, lane);
            __syncthreads();
        }
    }

    // general pair-point stepping (not FULL)
    const float invL = 1.0f / (float)L;
    const int l0 = FULL ? 0 : tid % L, m0 = FULL ? 0 : tid / L;
    const int dl = FULL ? 0 : G % L, dm = FULL ? 0 : G / L;

    // Each lane stands for one axis (lanes 1 .. DIM of each four; the others repeat an axis and are never
    // looked at). What it needs of it, relative to the anchor voxel where it is a place, lies in LDS: the
    // registers belong to the gathers. rec: 1/h, the volume's faces, h, the range that the box covers, the
    // axis's last voxel.
    float *rec = lds_axis + wave * 32 + (lane & 3) * 8;
    int anc[3] = {s.anc[0], s.anc[1], s.anc[2]};
    float off_l = (lane & 3) == 3 && DIM == 3 ? s.off[2] : ((lane & 3) == 2 ? s.off[1] : s.off[0]);
    long base = 0;
    Tile tile;
    tile.valid = false;
    float retry = 3.0e38f;     // no box fitted a ball this large: not tried again until it has shrunk or moved
    auto axis = [&](int t, int v0, int v1, int v2) {
        const int l = opaque(t) & 3;
        return DIM == 3 && l == 3 ? v2 : (l == 2 ? v1 : v0);
    };
    auto anchored = [&]() {
        const int al = axis(lane, anc[0], anc[1], anc[2]);
        rec[1] = (float)(-al);
        rec[2] = (float)(__float_as_int(rec[6]) - al);
        base = anc[0] + (long)anc[1] * vol.nx;
        if constexpr (DIM == 3) base += (long)anc[2] * vol.nxy;
        if constexpr (STAGE) {
            const int tl = axis(lane, tile.lo[0], tile.lo[1], tile.lo[2]);
            const int tn = axis(lane, tile.n[0], tile.n[1], tile.n[2]);
            // floor(v) >= lo and floor(v) + 1 < lo + n for whole lo and n
            rec[4] = tile.valid ? (float)(tl - al) : 3.0e38f;
            rec[5] = tile.valid ? (float)(tl + tn - 1 - al) : -3.0e38f;
        }
    };
    rec[0] = __int_as_float(axis(lane, __float_as_int(p.g.inv_h[0]), __float_as_int(p.g.inv_h[1]),
                                 __float_as_int(p.g.inv_h[2])));
    rec[3] = __int_as_float(axis(lane, __float_as_int(p.g.h[0]), __float_as_int(p.g.h[1]), __float_as_int(p.g.h[2])));
    rec[6] = __int_as_float(axis(lane, p.g.nx, p.g.ny, p.g.nz) - 1);
    anchored();
    float R = s.R;
    int status = s.status;
    int streak = s.streak;
    float e_mc = s.e_mc;
    const float inv_npts = uni<G>(1.0f / (float)(p.M * p.L));
    const float tol2 = uni<G>(p.conv_tol * p.conv_tol);
    int cull_next = p.cull_first;  // this launch's next culling pass point (-1: none)
    int blk = 0, sl = 0;
    int rot_next = EXACT || nb == 1 ? 0 : dr.K;   // the next block's entries in the set of rotations

    int it = 0;
    for (; it < budget && (status & 0x0f) == SNK_ACTIVE; ++it) {
        // no multiply-add contraction: every instance (with or without the optional terms below) rounds
        // the step operation by operation, so their results agree bit for bit
#pragma clang fp contract(off)
        const int gl = opaque(tid);
        const int lane = gl & 63;
        Frame<DIM> fr;
        const float smax_v = R + 0.5f * p.dR;
        set_frame<DIM, G>(fr, p, uni<G>(smax_v), RHO * R, R);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            fr.anc[a] = anc[a];
            fr.off[a] = a < DIM ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(off_l), 1 + a)) : 0.0f;
        }
        fr.base = base;
        // clamping can be skipped when the whole sample ball (with a rounding margin) is interior
        const float4 r0 = *reinterpret_cast<const float4 *>(rec);
        const float ext = fmaf(smax_v * r0.x, 1.0001f, 1e-3f);
        const float below = off_l - ext, above = off_l + ext;
        const bool interior = (__builtin_amdgcn_ballot_w64(below > r0.y && above < r0.z) & AXES) == AXES;
        int nvol[3] = {0, 0, 0};
        if (!interior) {
            const Cold<JobParams> q = cold(cp);
            nvol[0] = q->g.nx;
            nvol[1] = q->g.ny;
            nvol[2] = q->g.nz;
        }
        // x: the totals of A, x, y, z (2D: A, x, y, B_R) in lanes 0 .. 3 of each four; br: B_R in every lane
        float x = 0.0f, br = 0.0f;
        auto reduce = [&](const float *acc) {
            const float v[5] = {acc[0], acc[3], acc[2], DIM == 3 ? acc[NR - 1] : acc[1], acc[1]};
            wave_quads<NR>(v, x, br);
        };
        float *red = lds_red + (it & 1) * 8 * PARTS;
        if constexpr (EXACT) {
            float acc[NR];
#pragma unroll
            for (int k = 0; k < NR; ++k) acc[k] = 0.0f;
            const float inv_h[3] = {p.g.inv_h[0], p.g.inv_h[1], p.g.inv_h[2]};
            const float hh[3] = {p.g.h[0], p.g.h[1], p.g.h[2]};
            if (interior)
                lattice_sums<DIM, G, false, LAYOUT>(vol, nvol, fr, hh, inv_h, gl, acc);
            else
                lattice_sums<DIM, G, true, LAYOUT>(vol, nvol, fr, hh, inv_h, gl, acc);
            reduce(acc);
        } else {
            const float4 *pu = dr.pu + ((blk & 1) * dr.K + sl) * MH;
            bool staged = false;
            if constexpr (STAGE) {
                if (interior) {
                    const float2 r1 = *reinterpret_cast<const float2 *>(rec + 4);
                    staged = (__builtin_amdgcn_ballot_w64(below >= r1.x && above < r1.y) & AXES) == AXES;
                    if (!staged && fr.smax < retry) {
                        const Cold<JobParams> q = cold(cp);
                        const float inv_h[3] = {q->g.inv_h[0], q->g.inv_h[1], q->g.inv_h[2]};
                        const int nv[3] = {q->g.nx, q->g.ny, q->g.nz};
                        int lo[3], hi[3];
                        ball_range<DIM>(fr, inv_h, lo, hi);
                        if (choose_tile<DIM>(lo, hi, nv, tile_cap, tile)) {
                            // the previous iteration's reads of the box ended at its reduction barrier
                            stage_tile<PG>(lds_tile, q->g.J, vol.nx, vol.nxy, tile, gl);
                            __syncthreads();
                            staged = true;
                            retry = 3.0e38f;
                        } else {
                            // 1/20 of the finest voxel smaller, or at another voxel
                            retry = fr.smax - 0.05f * __builtin_amdgcn_rcpf(fmaxf(inv_h[0], fmaxf(inv_h[1], DIM == 3 ? inv_h[2] : 0.0f)));
                        }
                        anchored();
                    }
                }
            }
#pragma unroll 1
            for (int part = 0; part < PARTS / WAVES; ++part) {
                const int sg = gl + part * PG;   // the lane of the group whose pair-points these are
                float acc[NR];
#pragma unroll
                for (int k = 0; k < NR; ++k) acc[k] = 0.0f;
                if (staged) {
                    TileVol<DIM> tv;
                    tv.t = lds_tile;
                    tv.nx = tile.n[0];
                    tv.nxy = tile.n[0] * tile.n[1];
                    Frame<DIM> ft = fr;
                    ft.base = (anc[0] - tile.lo[0]) + (anc[1] - tile.lo[1]) * tv.nx;
                    if constexpr (DIM == 3) ft.base += (anc[2] - tile.lo[2]) * tv.nxy;
                    lane_sums<DIM, G, U, false, GRADI, FULL>(tv, nvol, ft, pu, P, L, invL, sg, l0, m0, dl, dm, acc);
                } else if (interior) {
                    lane_sums<DIM, G, U, false, GRADI, FULL>(vol, nvol, fr, pu, P, L, invL, sg, l0, m0, dl, dm, acc);
                } else {
                    lane_sums<DIM, G, U, true, GRADI, FULL>(vol, nvol, fr, pu, P, L, invL, sg, l0, m0, dl, dm, acc);
                }
                reduce(acc);
                if constexpr (PG < G) {
                    if (lane < 5) red[(wave + part * WAVES) * 8 + lane] = (DIM == 3 && lane == 4) ? br : x;
                }
            }
        }
        // draws ahead
        typename WaveDraws<DIM, PG>::Pending pend;
        pend.on = false;
        if constexpr (!EXACT) {
            if (sl == 0 && it + dr.K < budget) {
                const int r = (wave + blk) & (WAVES - 1);
                if (r < dr.passes) pend = dr.begin(r, (uint32_t)(n0 + 1 + it + dr.K), id, cp, lane);
            }
        }

        const int n = n0 + it + 1;
        float smax_d = smax_v;
#pragma unroll
        for (int i = 1; i < DIM; ++i) smax_d *= smax_v;
        // Monte-Carlo: V/N; exact: the voxel measure
        const float scale = EXACT ? p.g.h[0] * p.g.h[1] * (DIM == 3 ? p.g.h[2] : 1.0f) : BALL * smax_d * inv_npts;
        const float inv2R = __builtin_amdgcn_rcpf(2.0f * R);
        float inv_norm = inv2R;
#pragma unroll
        for (int i = 1; i < DIM; ++i) inv_norm *= inv2R;
        const float eps = p.eps0 * __builtin_amdgcn_rsqf((float)n);
        const float half_eps = 0.5f * eps;
        const float kc = -half_eps * scale * inv_norm;
        if constexpr (PARTS > 1) {
            // per-wave partials, added in wave order by every wave, so all of them hold the same totals
            // and take the same step (no second barrier to hand one wave's result to the others)
            if constexpr (PG == G) {
                if (lane < 5) red[wave * 8 + lane] = (DIM == 3 && lane == 4) ? br : x;
            }
            __syncthreads();
            x = red[lane & 3];
            if constexpr (DIM == 3) br = red[4];
#pragma unroll
            for (int w = 1; w < PARTS; ++w) {
                x += red[w * 8 + (lane & 3)];
                if constexpr (DIM == 3) br += red[w * 8 + 4];
            }
        }
        if constexpr (DIM == 2) br = dpp<0xFF>(x);   // quad_perm [3, 3, 3, 3]
        const float a0 = dpp<0x00>(x);               // quad_perm [0, 0, 0, 0]
        // gradient form: sum S dI/dv_a (voxel coordinates) -> the units of the weight form's
        // sum -dS/dr I u_a / h_a, i.e. the physical force divided by h_a
        const float4 r2 = *reinterpret_cast<const float4 *>(rec);   // 1/h, faces, h
        if constexpr (GRADI) x *= r2.x * r2.x;

        // descent step: radius and energy in every lane, each axis of the centre in its lanes
        const float A = scale * a0;
        const float BR = scale * br;
        const float E = A * inv_norm;
        const float gR = (BR - (2.0f * DIM) * inv2R * A) * inv_norm;
        float dRs = -half_eps * gR;
        float doff = kc * x;   // voxel units (B_c was accumulated against u / h)
        float dc = doff * r2.w;
        if (rp.cnt >= 0) {
            const Cold<EvolveArgs> ra = cold(rp.a);
            // repulsion of the neighbours' snapshot: lane k takes neighbour k; with t = |c - c_j| /
            // (rho (R + R_j)) < 1 the penalty (1 - t)^2 has dP/dc = -2 (1 - t) (c - c_j) /
            // (|c - c_j| rho (R + R_j)) and dP/dR = 2 (1 - t) t / (R + R_j)
            float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // R, y, x, z: totals in lanes R, x, y, z
            if (lane < rp.cnt) {
                const int j = ra->nb[(long)rp.cid * ra->nb_cap + lane];
                const float4 s0 = ra->snap[2 * j], s1 = ra->snap[2 * j + 1];
                const int aj[3] = {__float_as_int(s0.x), __float_as_int(s0.y), __float_as_int(s0.z)};
                const float oj[3] = {s1.x, s1.y, s1.z};
                float dv[3] = {0.0f, 0.0f, 0.0f}, d2 = 0.0f;
#pragma unroll
                for (int a = 0; a < DIM; ++a) {
                    dv[a] = ((float)(anc[a] - aj[a]) + (fr.off[a] - oj[a])) * ra->p.g.h[a];
                    d2 = fmaf(dv[a], dv[a], d2);
                }
                const float d = __builtin_amdgcn_sqrtf(d2);
                const float span = RHO * (R + s0.w);
                const float t = d / span;
                if (t < 1.0f) {
                    const float om = 1.0f - t;
                    v[0] = 2.0f * om * t / (R + s0.w);
                    if (d > 0.0f) {
                        const float f = -2.0f * om / (d * span);
                        v[2] = f * dv[0];
                        v[1] = f * dv[1];
                        v[3] = f * dv[2];
                    }
                }
            }
            float rt, unused;
            wave_quads<4>(v, rt, unused);
            const float kr = -half_eps * ra->kappa;
            dRs = dRs + kr * dpp<0x00>(rt);
            const float dcr = kr * rt;
            dc = dc + dcr;
            doff = doff + dcr * r2.x;
        }
        // |dc|^2 in axis order: lane 1 + i adds its square to lane i's sum
        const float q1 = dc * dc;
        float dc2 = fmaf(dc, dc, dpp<0x90>(q1));                        // quad_perm [0, 0, 1, 2]: lane 2 x, y
        if constexpr (DIM == 3) dc2 = fmaf(dc, dc, dpp<0x90>(dc2));     // lane 3 x, y, z
        if (TRACE && gl < 4) {
            float *row = trace_row;
            if (gl == 0) {
                row[0] = A;
                row[1] = BR;
                row[5] = E;
                row[6] = dRs;
                row[10] = (float)n;
                row[11] = R;
                row[12] = eps;
                row[13] = row[14] = row[15] = 0.0f;
            } else {
                row[1 + gl] = gl <= DIM ? scale * x * r2.w : 0.0f;
                row[6 + gl] = gl <= DIM ? dc : 0.0f;
            }
        }
        float Rn = R + dRs;
        int flag = status & SNK_CLAMPED;
        if (__builtin_amdgcn_ballot_w64(Rn < p.r_lo || Rn > p.r_hi) != 0) {
            if (Rn < p.r_lo) Rn = p.r_lo;
            if (Rn > p.r_hi) Rn = p.r_hi;
            flag = SNK_CLAMPED;
        }
        const float dRe = Rn - R;
        const bool small = (__builtin_amdgcn_ballot_w64(dRe * dRe < tol2 && dc2 < tol2) & LAST) != 0;
        R = Rn;
        e_mc = uni<G>(E);
        off_l += doff;
        int st = SNK_ACTIVE;
        const bool finite_l = isfinite(Rn) && isfinite(E);
        // a new anchor voxel, beyond a face, or not finite: seldom
        if ((__builtin_amdgcn_ballot_w64(!(fabsf(off_l) < 0.5f) || off_l < r2.y || off_l > r2.z || !finite_l) & AXES) !=
            0) {
            if ((__builtin_amdgcn_ballot_w64(!finite_l || !isfinite(off_l)) & AXES) != 0) {
                st = SNK_NONFINITE;
            } else {
                const bool far = fabsf(off_l) >= 0.5f;
                const float k = far ? rintf(off_l) : 0.0f;
                if (far) off_l -= k;
#pragma unroll
                for (int i = 0; i < DIM; ++i) anc[i] += __builtin_amdgcn_readlane((int)k, 1 + i);
                anchored();
                retry = 3.0e38f;
                if ((__builtin_amdgcn_ballot_w64(off_l < rec[1] || off_l > rec[2]) & AXES) != 0) st = SNK_OUT;
            }
        }
        if (st == SNK_ACTIVE) {
            streak = small ? min(streak + 1, 255) : 0;
            if (p.conv_window > 0 && streak >= p.conv_window) st = SNK_CONVERGED;
        }
        // a culling pass without competition judges each contour alone: at the run's pass points an
        // active contour above the threshold retires here and frees its slot at once (the pass after
        // the evolution treats the others as the passes between chunks would)
        if (it == cull_next) {
            const Cold<JobParams> q = cold(cp);
            if (st == SNK_ACTIVE && __builtin_amdgcn_ballot_w64(!(E <= q->cull_thr)) != 0) st = SNK_CULLED;
            cull_next = cull_next + q->cull_every <= q->cull_last ? cull_next + q->cull_every : -1;
        }
        status = st | flag;
        if constexpr (!EXACT) {
            if (sl == 0 && it + dr.K < budget) {
                dr.finish(pend, (blk + 1) & 1, rot_next, cp);
                // blocks of more passes than waves
                for (int r = ((wave + blk) & (WAVES - 1)) + WAVES; r < dr.passes; r += WAVES)
                    dr.finish(dr.begin(r, (uint32_t)(n0 + 1 + it + dr.K), id, cp, lane), (blk + 1) & 1, rot_next, cp);
            }
            if (++sl == dr.K) {
                sl = 0;
                if ((blk + 2) % nb == 0 && wave == ((blk + 2) / nb & (WAVES - 1)))
                    dr.rotations((uint32_t)(n0 + 2 + it + dr.K), id, cp, lane);
                ++blk;
                rot_next = rot_next + dr.K == dr.KR ? 0 : rot_next + dr.K;
            }
        }
        // one wave's LDS operations complete in order: only the compiler must keep them so
        if constexpr (WAVES == 1) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }

    float off_out[3] = {s.off[0], s.off[1], s.off[2]};
#pragma unroll
    for (int i = 0; i < DIM; ++i) off_out[i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(off_l), 1 + i));
    if (tid == 0) {
        DevContour o = s;
        for (int i = 0; i < 3; ++i) {
            o.anc[i] = anc[i];
            o.off[i] = off_out[i];
        }
        o.R = R;
        o.e_mc = e_mc;
        o.iters = n0 + it;
        o.status = (uint8_t)status;
        o.streak = (uint8_t)streak;
        *slot = o;
        atomicAdd(counter, (unsigned long long)it);
    }
}

// LDS of a sub-wave workgroup: the draws of each contour it holds.
template <int G>
__host__ __device__ __forceinline__ int sub_lds_floats(int MH) {
    return Grp<G>::CPB * ((draw_floats(G, MH) + 3) & ~3);
}

// Waves per SIMD asked of the compiler (1: its choice), the most that spill no vector register. One pair-point in
// flight: 2D 64 registers, 8 waves; 3D 74, 6 waves, and 85 with a box, 5 (at 8 waves up to 38 spilled: 2,000 contours,
// 128 lanes, 30 iterations with a box 274 us, now 230; 256 lanes 308, now 221). FULL 3D instances with two in flight
// and no box: 93 registers, 5 waves (98 and 4 waves unasked; lattice 10.6 ms against 10.9). In 2D the compiler's 86
// registers (5 waves) are the best: 6 or 7 waves spill nothing but put more contours' footprints in the L2 than it
// holds (8192^2 image 5.1 ms; 7 waves 5.3, 8 waves 6.2; 4 waves, held by LDS, 5.4). Two-wave groups with four
// in flight: 2D 114 registers, 4 waves; 3D 163, 3 waves (2,000 contours with a box 279 -> 230 us), but 4 where pairs or
// quads are gathered without a box, so that 8 contours per CU stay resident: 14 spilled (251 us, 266 at 3 waves). With
// a box and two in flight the LDS holds 8 contours of two waves per CU, so registers are left alone (109).
template <int DIM, int G, int U, int LAYOUT, bool STAGE, bool GRADI, bool FULL>
constexpr int waves_asked() {
    if (G < 64) return 1;
    if (U == 1) return DIM == 2 ? 8 : (STAGE ? 5 : 6);
    if (U == 4) return G != 128 ? 1 : (DIM == 2 || (!STAGE && (LAYOUT == kBufferPair || LAYOUT == kBufferQuad)) ? 4 : 3);
    return DIM == 3 && FULL && !STAGE && !GRADI ? 5 : 1;
}

// STAGE: the workgroup's LDS ends with a box of a.tile_cap voxels. GRADI: centre force in its
// image-gradient form. FULL: L = 16 and whole passes (full_passes).
// PG: lanes of the workgroup (whole-wave groups: see run_wave).
template <int DIM, int G, int U, bool TRACE, int LAYOUT, bool EXACT, bool STAGE, bool GRADI, bool FULL,
          int PG = Grp<G>::NT>
__global__ __launch_bounds__(PG, (waves_asked<DIM, G, U, LAYOUT, STAGE, GRADI, FULL>()))
void evolve_kernel(EvolveArgs a) {
    extern __shared__ __align__(16) float lds[];
    if constexpr (G < 64) {
        const int per = (draw_floats(G, a.p.M / 2) + 3) & ~3;
        const int sub = (int)threadIdx.x / G;
        const int k = blockIdx.x * Grp<G>::CPB + sub;
        const int cid = k < a.n ? (a.idx ? a.idx[k] : k) : k;
        DevContour *slot = k < a.n ? a.st + cid : nullptr;
        run_group<DIM, G, U, TRACE, LAYOUT, EXACT>(a.p, slot, a.n_iter,
                                                   TRACE && slot ? a.trace + (long)cid * SNK_TRACE_W : nullptr,
                                                   lds + sub * per, a.counter);
    } else {
        const int cid = a.idx ? __builtin_amdgcn_readfirstlane(a.idx[blockIdx.x]) : (int)blockIdx.x;
        // the arguments where the launch put them (EvolveArgs is the kernel's only argument, p its first member)
        const Cold<EvolveArgs> ca = (Cold<EvolveArgs>)__builtin_amdgcn_kernarg_segment_ptr();
        Repel rp{ca, cid, -1};
        if (a.kappa > 0.0f) rp.cnt = __builtin_amdgcn_readfirstlane(a.nbn[cid]);
        run_wave<DIM, G, U, TRACE, LAYOUT, EXACT, STAGE, GRADI, FULL, PG>(
            a.p, (Cold<JobParams>)ca, a.st + cid, a.n_iter, 0x7fffffff,
            TRACE ? a.trace + (long)cid * SNK_TRACE_W : nullptr, lds, a.draw_k, a.rot_k, a.counter,
            STAGE ? a.tile_cap : 0, rp);
    }
}

template <int DIM, int G, int U, bool TRACE, int LAYOUT, bool EXACT, bool STAGE, bool GRADI, bool FULL,
          int PG = Grp<G>::NT>
hipError_t launch_f(EvolveArgs a, hipStream_t s) {
    size_t lds;
    if constexpr (G >= 64) {
        const DrawPlan d = draw_plan(DIM, a.p.M / 2, STAGE);
        a.draw_k = d.K;
        a.rot_k = d.KR;
        lds = wave_lds_bytes(G, PG, EXACT ? 0 : wave_draw_floats(DIM, d.K, d.KR, a.p.M / 2), STAGE ? a.tile_cap : 0);
    } else {
        lds = sizeof(float) * (size_t)sub_lds_floats<G>(a.p.M / 2);
    }
    const int blocks = (a.n + Grp<G>::CPB - 1) / Grp<G>::CPB;
    hipLaunchKernelGGL((evolve_kernel<DIM, G, U, TRACE, LAYOUT, EXACT, STAGE, GRADI, FULL, PG>), dim3(blocks),
                       dim3(PG), lds, s, a);
    return hipGetLastError();
}

// FULL instances where the sampling allows (they exist outside the per-iteration trace, whose sums have the
// same order).
template <int DIM, int G, int U, bool TRACE, int LAYOUT, bool EXACT = false, bool STAGE = false, bool GRADI = false>
hipError_t launch_t(const EvolveArgs &a, hipStream_t s) {
    if constexpr (G >= 64 && U >= 2 && !TRACE && !EXACT)
        if (full_passes(G, U, a.p.M, a.p.L)) {
            // two waves do the work of four where the launch shape says so (mc_shape)
            if constexpr (DIM == 3 && G == 256 && STAGE && !GRADI && LAYOUT != kBufferQuad)
                if (a.two_waves)
                    return launch_f<DIM, G, U, TRACE, LAYOUT, EXACT, STAGE, GRADI, true, 128>(a, s);
            return launch_f<DIM, G, U, TRACE, LAYOUT, EXACT, STAGE, GRADI, true>(a, s);
        }
    return launch_f<DIM, G, U, TRACE, LAYOUT, EXACT, STAGE, GRADI, false>(a, s);
}

}  // namespace

}  // namespace snk
