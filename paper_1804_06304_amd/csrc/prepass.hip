// Dispatch of the pre-pass to the kernels of its raw type (prepass_u8.hip, prepass_u16.hip, prepass_f32.hip),
// and the second copies of an existing smoothed volume.
#include <algorithm>

#include "snk_internal.h"

namespace snk {

namespace {

// Quad records of one row segment from an existing J: J(x,y), J(x+1,y), J(x,y+1), J(x+1,y+1) of
// plane z, the neighbours clamped to the last column / row (only cells with x <= nx-2, y <= ny-2 are
// gathered).
__global__ __launch_bounds__(256) void pack_quad_kernel(const float *__restrict__ J, float4 *__restrict__ Jq,
                                                       int nx, int ny, int nz) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    const int z = blockIdx.z;
    if (x >= nx) return;
    const long row = ((long)z * ny + y) * nx;
    const long row1 = ((long)z * ny + min(y + 1, ny - 1)) * nx;
    const int x1 = min(x + 1, nx - 1);
    Jq[row + x] = make_float4(J[row + x], J[row + x1], J[row1 + x], J[row1 + x1]);
}

}  // namespace

hipError_t launch_pack_quad(const float *J, float4 *Jq, int nx, int ny, int nz, hipStream_t s) {
    if (nx <= 0 || ny <= 0 || nz <= 0) return hipSuccess;
    if (ny > 65535 || nz > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(pack_quad_kernel, dim3((nx + 255) / 256, ny, nz), dim3(256), 0, s, J, Jq, nx, ny, nz);
    return hipGetLastError();
}

namespace {
// Column pairs of a 2D image: Jp[y][x] = (J[y][x], J[y + 1][x]), the last row paired with itself.
__global__ __launch_bounds__(256) void pack_pair_kernel(const float *__restrict__ J, float2 *__restrict__ Jp,
                                                        int nx, int ny) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    const long plane = (long)blockIdx.z * ny * nx;
    if (x >= nx) return;
    const long row = plane + (long)y * nx, row1 = plane + (long)min(y + 1, ny - 1) * nx;
    Jp[row + x] = make_float2(J[row + x], J[row1 + x]);
}
}  // namespace

hipError_t launch_pack_pair(const float *J, float2 *Jp, int nx, int ny, int nz, hipStream_t s) {
    if (nx <= 0 || ny <= 0 || nz <= 0) return hipSuccess;
    hipLaunchKernelGGL(pack_pair_kernel, dim3((nx + 255) / 256, ny, nz), dim3(256), 0, s, J, Jp, nx, ny);
    return hipGetLastError();
}

int prepass_rows_per_thread(const PrepassArgs &a) { return a.rz <= 8 ? 4 : 2; }

namespace {
hipError_t launch_typed(const PrepassJob &one, const PrepassJob *jobs, int n, int blocks, hipStream_t s, int *slots) {
    switch (one.a.dtype) {
        case SNK_U8: return launch_prepass_u8(one, jobs, n, blocks, s, slots);
        case SNK_U16: return launch_prepass_u16(one, jobs, n, blocks, s, slots);
        default: return launch_prepass_f32(one, jobs, n, blocks, s, slots);
    }
}
}  // namespace

// Whether workgroups march down an image's rows of tiles (prepass_tile): by chunks of six, for all but 32-bit images
// written in pairs by the kernel of radius 3, bound by memory (march, a tile each: 8,192^2 u8, sigma 0 / 1 / 3: 111 / 108
// / 419 us, 171 / 155 / 476; 60,000 x 64 15 / 14 / 38, 17 / 16 / 38; pairs, sigma 1: 8,192^2 u8 210, 248, f32 234, 231;
// 4,096^2 u8 49, 51, f32 62, 51).
bool prepass_marches(const PrepassArgs &a) {
    return a.nz == 1 && !a.Jq && !(a.Jp && a.dtype == SNK_F32 && a.rx == 3 && a.ry == 3);
}

// A workgroup's chunk of z planes (an image's rows of tiles) takes 2 rz more to fill its ring, so small chunks are more
// work, and large ones leave the chip idle. A plane takes a CU some 6 + w units with w workgroups on it (512 x 512
// planes, radius 3: 1.35 us alone, 2.1 with two, 3.6 with six), so the chunk is the one of least (chunk + 2 rz + 2) times
// that, summed over the rounds of resident workgroups (411 x 387 x 131, sigma 1.6: 5 chunks, one round, 139 us; 6
// chunks, a little more than a round, 164; 64^3, sigma 1.6 / 3 / 5.3: chunks of 5 / 9 / 16 planes 41 / 135 / 397 us, of
// 1 / 2 / 2 31 / 101 / 275). Where no ring is to be filled chunks are short, and several rounds even out (at most 6:
// 8,192^2 u8, sigma 1, 32 rows of tiles 122 us, 6 103; u16 with pairs, sigma 1.6, 37 rows 310, 6 259; 512 x 512 x 128
// unsmoothed with quads, 22 planes 160, 6 145).
int prepass_plan(PrepassJob *jobs, int n, int cus, int lds_per_cu) {
    if (n <= 0) return 0;
    const int ty = 4 * prepass_rows_per_thread(jobs[0].a), tx = jobs[0].a.Jq ? 63 : 64;
    int top = 0;
    for (int i = 0; i < n; ++i) {
        PrepassJob &j = jobs[i];
        const int rows = (j.a.ny + ty - 1) / ty;
        const bool march = prepass_marches(j.a);
        j.cut.bx = (j.a.nx + tx - 1) / tx;
        j.cut.by = march ? 1 : rows;
        j.cut.len = march ? rows : j.a.nz;
        top = std::max(top, j.cut.len);
    }
    // (a device that did not say: a whole chip's)
    if (cus <= 0) cus = 256;
    int per_cu = lds_per_cu > 0 ? lds_per_cu : 160 * 1024;
    (void)launch_typed(jobs[0], nullptr, 0, 0, nullptr, &per_cu);
    const long slots = (long)per_cu * cus;
    const int rz = jobs[0].a.rz;
    auto groups_of = [](const PrepassJob &j, int chunk) {
        return (long)j.cut.bx * j.cut.by * ((j.cut.len + chunk - 1) / chunk);
    };
    int chunk = top;
    double best = 0.0;
    // (the chunk lengths that cut `top` evenly, longest first; the stream may be idle meanwhile)
    for (int z = top;;) {
        long groups = 0;
        for (int i = 0; i < n; ++i) groups += groups_of(jobs[i], z);
        const long rest = groups % slots;
        const double round = (double)(groups / slots) * (6.0 + per_cu) +
                             (rest ? 6.0 + std::max(1.0, (double)rest / cus) : 0.0);
        const double cost = round * (z + 2 * rz + 2);
        if (z == top || cost < best) {
            best = cost;
            chunk = z;
        }
        if (z == 1 || groups > 4 * slots) break;
        const int c = (top + z - 2) / (z - 1);   // the fewest chunks of less than z
        z = (top + c - 1) / c;
    }
    if (rz == 0) chunk = std::min(chunk, std::max(6, (top + 65534) / 65535));   // (a grid has 65,535 chunks)
    int first = 0;
    for (int i = 0; i < n; ++i) {
        PrepassJob &j = jobs[i];
        j.first = first;
        const int k = (j.cut.len + chunk - 1) / chunk;
        j.cut.chunk = (j.cut.len + k - 1) / k;
        first += (int)groups_of(j, j.cut.chunk);
    }
    return first;
}

hipError_t launch_prepass(const PrepassArgs &a, int cus, int lds_per_cu, hipStream_t s) {
    PrepassJob one{};
    one.a = a;
    const int blocks = prepass_plan(&one, 1, cus, lds_per_cu);
    return launch_typed(one, nullptr, 0, blocks, s, nullptr);
}

bool prepass_same_launch(const PrepassArgs &a, const PrepassArgs &b) {
    return a.dtype == b.dtype && a.rx == b.rx && a.ry == b.ry && a.rz == b.rz && !a.Jq == !b.Jq && !a.Jp == !b.Jp &&
           prepass_marches(a) == prepass_marches(b);
}

hipError_t launch_prepass_batch(const PrepassJob *host, const PrepassJob *dev, int n, int blocks, hipStream_t s) {
    if (n <= 0 || blocks <= 0) return hipSuccess;
    return launch_typed(host[0], dev, n, blocks, s, nullptr);
}

}  // namespace snk
