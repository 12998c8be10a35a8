// Pre-pass: affine intensity map and separable Gaussian low-pass (the paper's low-pass filter that
// keeps Monte-Carlo integration well behaved, Sec. II-E), clamp-to-edge, raw u8/u16/f32 -> FP32,
// optionally also written as quad records or column pairs. The kernels of one raw type, instantiated in
// prepass_u8.hip, prepass_u16.hip and prepass_f32.hip.
//
// A workgroup of 64 columns x 4 row groups evaluates a tile of 64 x 4 ROWS and marches along a chunk of z.
// Per input plane: stage the plane with its x/y halo in LDS from registers that were fetched while the
// previous plane was filtered; barrier; filter along x into LDS; barrier; then every thread filters its own
// ROWS neighbouring rows of one column along y (from the 2 ry + ROWS values they share) and z (a ring of
// 2 rz + 1 planes of its own rows, in its registers), and stores J and the second copy. A column pair's lower row
// is a row that the thread evaluates too (one more than it stores); a quad record's +x values come from the next
// lane, so tiles are 63 columns wide there and 64, whole cache lines, otherwise.
//
// Small radii are bound by HBM (raw read, 4 B of J and 8 B of pairs or 16 B of quads per voxel), larger ones by
// the latency of a plane's two barriers and LDS reads. A thread's rows lie next to each other because they share
// their column's values, the ring is in registers because LDS rings left two workgroups on a CU, and nothing is
// read back to find a neighbour. Against rows 4 apart, their ring in LDS and the filtered plane exchanged through
// it (411 x 387 x 131 f32 with pairs, sigma 1.6: 460 -> 148 us; 384 x 384 x 96 u8 with pairs, sigma 1 / 1.6 / 2.6 /
// 5.3: 80 / 388 / 430 / 1,889 -> 56 / 96 / 195 / 953 us; 4096^2 u8 alone, sigma 1 / 1.6: 44 / 135 -> 35 / 52 us).
// Sums kept per output instead of a ring (no moves) measured the same: the moves are hidden.
#pragma once

#include <algorithm>
#include <type_traits>

#include "snk_internal.h"

namespace snk {

namespace {

constexpr int EX = 64;     // columns evaluated per tile, one per lane
constexpr int NT = 256;
constexpr int GROUPS = NT / EX;

// Arguments in constant memory: the taps are scalar loads.
typedef const __attribute__((address_space(4))) PrepassArgs *ArgsPtr;

typedef const __attribute__((address_space(4))) float *TapsPtr;
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));

// f(integral_constant) of a radius known when the kernel runs: 0 .. 8 unrolled, -1 beyond (of kernels that take more).
template <int RXY, int RB, typename F>
__device__ __forceinline__ void with_radius(int r, F f) {
    if constexpr (RXY >= 0) {
        f(std::integral_constant<int, RXY>());
    } else {
        switch (r) {
            case 0: return f(std::integral_constant<int, 0>());
            case 1: return f(std::integral_constant<int, 1>());
            case 2: return f(std::integral_constant<int, 2>());
            case 3: return f(std::integral_constant<int, 3>());
            case 4: return f(std::integral_constant<int, 4>());
            case 5: return f(std::integral_constant<int, 5>());
            case 6: return f(std::integral_constant<int, 6>());
            case 7: return f(std::integral_constant<int, 7>());
            case 8: return f(std::integral_constant<int, 8>());
            default:
                if constexpr (RB > 8) return f(std::integral_constant<int, -1>());
        }
    }
}

// One value filtered along x: sum over the 2 R + 1 taps, in tap order.
template <int R>
__device__ __forceinline__ float filter_row(TapsPtr g, const float *row) {
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k <= 2 * R; ++k) acc = fmaf(g[k], row[k], acc);
    return acc;
}

// N neighbouring values of a column filtered along y, each in tap order, from the N + 2 r values they share.
template <int R, int N>
__device__ __forceinline__ void filter_column(TapsPtr g, int r, const float *col, float *v) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = 0.0f;
    if constexpr (R >= 0) {
        float c[N + 2 * R];
#pragma unroll
        for (int i = 0; i < N + 2 * R; ++i) c[i] = col[i * EX];
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int k = 0; k <= 2 * R; ++k) v[i] = fmaf(g[k], c[i + k], v[i]);
    } else {
        float c[N];
#pragma unroll
        for (int i = 0; i + 1 < N; ++i) c[i] = col[i * EX];
#pragma unroll 4
        for (int k = 0; k <= 2 * r; ++k) {
            c[N - 1] = col[(k + N - 1) * EX];
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = fmaf(g[k], c[i], v[i]);
#pragma unroll
            for (int i = 0; i + 1 < N; ++i) c[i] = c[i + 1];
        }
    }
}

// The tile's part of a row of a copy: a lane past its bytes stores nothing. With the bounds in the descriptor and
// not in branches every plane issues the same stores, so the wait for the next plane's loads, which were issued
// before them and share their counter, need not drain them.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(void *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x00027000);
}

// SECOND: also write the quad records (1) or the column pairs (2). RXY >= 0: the x and y radius is a
// compile-time constant; -1: at most RB, from the arguments. RZ: the z radius, or with ZMAX the largest one,
// the radius being the arguments'.
template <int SECOND>
constexpr int tile_columns() {
    return SECOND == 1 ? EX - 1 : EX;
}
template <int ROWS, int SECOND>
constexpr int rows_evaluated() {
    return ROWS + (SECOND ? 1 : 0);
}

// Tile (bx, by) of the planes z0 .. z1 - 1 of volume a; with MARCH, of an image (nz = 1) the tiles (bx, z0 .. z1 - 1),
// which a workgroup marches over as it does over planes, its next loads in flight (8192^2 u8 alone 155 -> 127
// us, 106 by chunks of six; never with quad records, 4096^2 71 -> 91, whose rows fall on the same channels).
template <typename T, int ROWS, int RXY, int RB, int RZ, bool ZMAX, int SECOND, bool MARCH>
__device__ __forceinline__ void prepass_tile(ArgsPtr a, int bx, int by, int z0, int z1, float *lds) {
    constexpr int EV = rows_evaluated<ROWS, SECOND>();
    constexpr int TX = tile_columns<SECOND>();
    constexpr int TY = GROUPS * ROWS;
    constexpr int KR = 2 * RZ + 1;
    constexpr int EXTRA = SECOND ? 1 : 0;                       // the row below the tile
    constexpr int NRA = (TY + EXTRA + 2 * RB + GROUPS - 1) / GROUPS;  // plane rows per thread (upper bound)
    constexpr int NCA = (EX + 2 * RB + EX - 1) / EX;            // plane columns per thread (upper bound)
    const int rx = RXY >= 0 ? RXY : a->rx;
    const int ry = RXY >= 0 ? RXY : a->ry;
    const int rz = ZMAX ? a->rz : RZ;
    const int PW = EX + 2 * rx;                  // plane row width
    const int PH = TY + EXTRA + 2 * ry;          // plane rows
    const int nx = a->nx, ny = a->ny, nz = a->nz;
    float *plane = lds;                          // PH x PW
    float *tmp = plane + PH * PW;                // PH x EX (x-filtered)
    float rr[EV][KR];                            // the ring: the last is the newest plane
#pragma unroll
    for (int i = 0; i < EV; ++i)
#pragma unroll
        for (int k = 0; k < KR; ++k) rr[i][k] = 0.0f;

    const int x0 = bx * TX, y0 = by * TY;
    const int t = threadIdx.x;
    const int tx = t & (EX - 1);
    const int ty = __builtin_amdgcn_readfirstlane(t >> 6);   // row group: one wave
    const long nxy = (long)nx * ny;
    auto plane_of = [&](int zi) { return MARCH ? 0 : zi; };
    auto first_row = [&](int zi) { return MARCH ? zi * TY : y0; };
    const T *raw = static_cast<const T *>(a->raw);
    const float off = a->i_offset, scale = a->i_scale;

    // raw plane values of this thread (rows ty + 4 i, columns tx + 64 j), clamp-to-edge; kept raw and
    // unconverted until staged, and loaded without a branch (slots past the plane read a clamped, valid
    // address and are not stored), so the loads stay in flight while the current plane is filtered
    T pre[NRA][NCA];
    auto fetch = [&](int zi) {
        const long zoff = (long)min(max(plane_of(zi), 0), nz - 1) * nxy;
        const int top = first_row(zi) - ry;
#pragma unroll
        for (int i = 0; i < NRA; ++i) {
            const int r = min(ty + GROUPS * i, PH - 1);
            const T *row = raw + (zoff + (long)min(max(top + r, 0), ny - 1) * nx);
#pragma unroll
            for (int j = 0; j < NCA; ++j) {
                const int c = min(tx + EX * j, PW - 1);
                pre[i][j] = row[min(max(x0 + c - rx, 0), nx - 1)];
            }
        }
    };

    // plane zi (fetched while the one before was filtered) into LDS, the fetch of the next (always: past the
    // chunk it reads a clamped plane again), the x and y filters, and the ring's next entry
    auto filter_xy = [&](int zi) {
#pragma unroll
        for (int i = 0; i < NRA; ++i) {
            const int r = ty + GROUPS * i;
            if (r < PH) {
#pragma unroll
                for (int j = 0; j < NCA; ++j) {
                    const int c = tx + EX * j;
                    if (c < PW) plane[r * PW + c] = ((float)pre[i][j] - off) * scale;
                }
            }
        }
        __syncthreads();
        fetch(zi + 1);
        with_radius<RXY, RB>(rx, [&](auto R) {
            if constexpr (decltype(R)::value >= 0) {
#pragma unroll
                for (int i = 0; i < NRA; ++i) {
                    const int r = ty + GROUPS * i;
                    if (r < PH) tmp[r * EX + tx] = filter_row<decltype(R)::value>(a->gx, plane + r * PW + tx);
                }
            } else {
                // the thread's rows side by side: their reads are in flight together (a row past the plane sums its last)
                float acc[NRA];
                const float *row[NRA];
#pragma unroll
                for (int i = 0; i < NRA; ++i) {
                    acc[i] = 0.0f;
                    row[i] = plane + min(ty + GROUPS * i, PH - 1) * PW + tx;
                }
#pragma unroll 2
                for (int k = 0; k <= 2 * rx; ++k) {
                    const float g = a->gx[k];
#pragma unroll
                    for (int i = 0; i < NRA; ++i) acc[i] = fmaf(g, row[i][k], acc[i]);
                }
#pragma unroll
                for (int i = 0; i < NRA; ++i)
                    if (ty + GROUPS * i < PH) tmp[(ty + GROUPS * i) * EX + tx] = acc[i];
            }
        });
        // the plane is free for the next one's staging, and the filtered rows until the barrier after that
        __syncthreads();
        float v[EV];
        with_radius<RXY, RB>(ry, [&](auto R) {
            filter_column<decltype(R)::value, EV>(a->gy, ry, tmp + ty * ROWS * EX + tx, v);
        });
#pragma unroll
        for (int i = 0; i < EV; ++i) {
#pragma unroll
            for (int k = 0; k + 1 < KR; ++k) rr[i][k] = rr[i][k + 1];
            rr[i][KR - 1] = v[i];
        }
    };

    const int x = x0 + tx;
    fetch(z0 - rz);
    int zi = z0 - rz;
    for (; zi < z0 + rz; ++zi) filter_xy(zi);   // these only fill the ring
    for (; zi < z1 + rz; ++zi) {
        filter_xy(zi);
        // z filter over planes zo - rz .. zo + rz, oldest first
        const int zo = zi - rz;
        float f[EV];
#pragma unroll
        for (int i = 0; i < EV; ++i) f[i] = 0.0f;
#pragma unroll
        for (int k = 0; k < KR; ++k) {
            const int kt = ZMAX ? k - 2 * (RZ - rz) : k;
            if (!ZMAX || kt >= 0) {
#pragma unroll
                for (int i = 0; i < EV; ++i) f[i] = fmaf(a->gz[kt], rr[i][k], f[i]);
            }
        }
        float fx[EV];   // the +x neighbours (quad records), clamped at the volume's last column
        if constexpr (SECOND == 1) {
#pragma unroll
            for (int i = 0; i < EV; ++i) {
                const float n = __shfl_down(f[i], 1, 64);
                fx[i] = x + 1 < nx ? n : f[i];
            }
        }
        const int yt = first_row(zo) + ty * ROWS;
        const long o0 = plane_of(zo) * nxy + (long)yt * nx + x0;
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const int y = yt + i;
            const bool in = y < ny, last = y + 1 >= ny;
            const long o = in ? o0 + (long)i * nx : 0;
            const int cells = in ? min(nx - x0, TX) : 0;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f[i]), row_buffer(a->J + o, cells * 4), tx * 4, 0, 0);
            if constexpr (SECOND == 1) {
                // non-temporal: the quad records (4x the volume) are written past the caches, which
                // shortens the pre-pass and does not slow the evolution that gathers from them
                const u4v q = {__float_as_uint(f[i]), __float_as_uint(fx[i]), __float_as_uint(last ? f[i] : f[i + 1]),
                               __float_as_uint(last ? fx[i] : fx[i + 1])};
                __builtin_amdgcn_raw_buffer_store_b128(q, row_buffer(a->Jq + o, cells * 16), tx * 16, 0, 2);
            }
            if constexpr (SECOND == 2) {
                const u2v q = {__float_as_uint(f[i]), __float_as_uint(last ? f[i] : f[i + 1])};
                __builtin_amdgcn_raw_buffer_store_b64(q, row_buffer(a->Jp + o, cells * 8), tx * 8, 0, 0);
            }
        }
    }
}

size_t prepass_lds(int rows, int rx, int ry, bool second) {
    return sizeof(float) * (size_t)(GROUPS * rows + (second ? 1 : 0) + 2 * ry) * (EX + 2 * rx + EX);
}

// Workgroup b of a table belongs to the volume whose `first` is the last at or below b; without a table there is
// one volume, the first argument, read where the launch put it, and the grid is its cut.
template <typename T, int ROWS, int RXY, int RB, int RZ, bool ZMAX, int SECOND, bool MARCH>
__global__ __launch_bounds__(NT) void prepass_kernel(PrepassJob one, const PrepassJob *jobs, int n) {
    extern __shared__ float lds[];
    typedef const __attribute__((address_space(4))) PrepassJob *JobPtr;
    JobPtr j = (JobPtr)__builtin_amdgcn_kernarg_segment_ptr();
    int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    if (n > 0) {
        const JobPtr table = (JobPtr)jobs;
        const int b = bx;
        int lo = 0, hi = n - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (table[mid].first <= b) lo = mid;
            else hi = mid - 1;
        }
        j = table + lo;
        const int k = b - j->first;
        bx = k % j->cut.bx;
        by = k / j->cut.bx % j->cut.by;
        bz = k / j->cut.bx / j->cut.by;
    }
    const int z0 = bz * j->cut.chunk;
    prepass_tile<T, ROWS, RXY, RB, RZ, ZMAX, SECOND, MARCH>(&j->a, bx, by, z0, min(j->cut.len, z0 + j->cut.chunk), lds);
}

// Workgroups of a kernel that a CU holds, by its registers: a workgroup is one wave on each SIMD, which has 512
// registers per lane to give out in eights.
inline int groups_by_registers(const void *kernel) {
    hipFuncAttributes at{};
    if (hipFuncGetAttributes(&at, kernel) != hipSuccess || at.numRegs <= 0) {
        (void)hipGetLastError();   // the launch's own check follows
        return 4;
    }
    return std::max(1, std::min(8, 512 / ((at.numRegs + 7) & ~7)));
}

// The planned volume one, or with n > 0 the n of a table of which it is the first. With slots, the LDS of a CU, the
// workgroups that a CU holds in its place, and no launch.
template <typename T, int ROWS, int RXY, int RB, int RZ, bool ZMAX, int SECOND, bool MARCH = false>
hipError_t launch_k(const PrepassJob &one, const PrepassJob *jobs, int n, int blocks, hipStream_t s, int *slots) {
    const size_t lds = prepass_lds(ROWS, one.a.rx, one.a.ry, SECOND != 0);
    if (slots) {
        static const int per_cu =
            groups_by_registers(reinterpret_cast<const void *>(&prepass_kernel<T, ROWS, RXY, RB, RZ, ZMAX, SECOND, MARCH>));
        *slots = std::max(1, std::min(per_cu, (int)((size_t)*slots / lds)));
        return hipSuccess;
    }
    const dim3 grid = n > 0 ? dim3(blocks) : dim3(one.cut.bx, one.cut.by, blocks / (one.cut.bx * one.cut.by));
    hipLaunchKernelGGL((prepass_kernel<T, ROWS, RXY, RB, RZ, ZMAX, SECOND, MARCH>), grid, dim3(NT), lds, s, one, jobs, n);
    return hipGetLastError();
}

template <typename T, int ROWS, int RXY, int RB, int RZ, bool ZMAX = false>
hipError_t launch_s(const PrepassJob &one, const PrepassJob *jobs, int n, int blocks, hipStream_t s, int *slots) {
    if constexpr (RZ == 0)
        if (prepass_marches(one.a))
            return one.a.Jp ? launch_k<T, ROWS, RXY, RB, RZ, ZMAX, 2, true>(one, jobs, n, blocks, s, slots)
                            : launch_k<T, ROWS, RXY, RB, RZ, ZMAX, 0, true>(one, jobs, n, blocks, s, slots);
    if (one.a.Jq) return launch_k<T, ROWS, RXY, RB, RZ, ZMAX, 1>(one, jobs, n, blocks, s, slots);
    if (one.a.Jp) return launch_k<T, ROWS, RXY, RB, RZ, ZMAX, 2>(one, jobs, n, blocks, s, slots);
    return launch_k<T, ROWS, RXY, RB, RZ, ZMAX, 0>(one, jobs, n, blocks, s, slots);
}

// The radii of sigma_pre = 1 on unit (x, y) spacing with z spacing 1, 2 or a 2D image have their own
// instances; others up to 8 share those with the z radius. A ring of more than 8 planes to each side takes two
// rows per thread: four would be 165 registers of it.
template <typename T>
hipError_t launch_r(const PrepassJob &one, const PrepassJob *jobs, int n, int blocks, hipStream_t s, int *slots) {
    constexpr int B = kPrepassMaxR;
    const PrepassArgs &a = one.a;
    if (prepass_rows_per_thread(a) == 2) return launch_s<T, 2, -1, B, B, true>(one, jobs, n, blocks, s, slots);
    if (a.rx > 8 || a.ry > 8) {
        if (a.rz == 0) return launch_s<T, 4, -1, B, 0>(one, jobs, n, blocks, s, slots);
        return launch_s<T, 4, -1, B, 8, true>(one, jobs, n, blocks, s, slots);
    }
    if (a.rx == 3 && a.ry == 3) {
        if (a.rz == 2) return launch_s<T, 4, 3, 3, 2>(one, jobs, n, blocks, s, slots);
        if (a.rz == 3) return launch_s<T, 4, 3, 3, 3>(one, jobs, n, blocks, s, slots);
        if (a.rz == 0) return launch_s<T, 4, 3, 3, 0>(one, jobs, n, blocks, s, slots);
    }
    switch (a.rz) {
        case 0: return launch_s<T, 4, -1, 8, 0>(one, jobs, n, blocks, s, slots);
        case 1: return launch_s<T, 4, -1, 8, 1>(one, jobs, n, blocks, s, slots);
        case 2: return launch_s<T, 4, -1, 8, 2>(one, jobs, n, blocks, s, slots);
        case 3: return launch_s<T, 4, -1, 8, 3>(one, jobs, n, blocks, s, slots);
        case 4: return launch_s<T, 4, -1, 8, 4>(one, jobs, n, blocks, s, slots);
        case 5: return launch_s<T, 4, -1, 8, 5>(one, jobs, n, blocks, s, slots);
        case 6: return launch_s<T, 4, -1, 8, 6>(one, jobs, n, blocks, s, slots);
        default: return launch_s<T, 4, -1, 8, 8, true>(one, jobs, n, blocks, s, slots);
    }
}

}  // namespace

}  // namespace snk
