// Resampling of the parameters between hierarchical levels (Sec. IV, hierarchical
// formulation): the next level's grid and environment layers are filled from the current
// ones by linear interpolation at the new cell and texel centres.  One launch: the first
// workgroups fill the grid, the others the layers.  A thread fills kColumn voxels of a column in z,
// so that the bilinear sample of a source plane serves every voxel that needs it (at a doubled
// resolution each plane serves four): the gathers, not the 16 B written per voxel, were the bound.
// 64^3 to 128^3 with three layers of 128x64 to 256x128 (39.7 MB at all): 11.1 us a call, 3.6 TB/s; 16.3 us
// with one voxel per thread, 64-bit index arithmetic and a launch of its own for the layers.
#include "perf_internal.h"

namespace perf {
namespace {

// Source coordinate of destination cell j along an axis (cell-centred): clamped to the
// source's first and last centres, lower index at most n_src - 2.
__device__ __forceinline__ void lerp_clamped(int j, int n_src, int n_dst, int& i0, float& f) {
    float g = ((float)j + 0.5f) * (float)n_src / (float)n_dst - 0.5f;
    g = fminf(fmaxf(g, 0.0f), (float)(n_src - 1));
    i0 = min((int)g, n_src - 2);
    f = g - (float)i0;
}

// Periodic axis (azimuth): the lower index wraps.
__device__ __forceinline__ void lerp_periodic(int j, int n_src, int n_dst, int& i0, int& i1, float& f) {
    const float g = ((float)j + 0.5f) * (float)n_src / (float)n_dst - 0.5f;
    const float fl = floorf(g);
    f = g - fl;
    i0 = (int)fl;
    i0 = ((i0 % n_src) + n_src) % n_src;
    i1 = (i0 + 1 == n_src) ? 0 : i0 + 1;
}

constexpr int kBlockUp = 256, kColumn = 4;

__device__ __forceinline__ float4 mix(float4 a, float wa, float4 b, float wb) {
    return make_float4(wa * a.x + wb * b.x, wa * a.y + wb * b.y, wa * a.z + wb * b.z, wa * a.w + wb * b.w);
}

struct Level {
    int nx, ny, nz, w, h;
};

// Voxels (x, y, z0 .. z0 + kColumn - 1), (x, y) = the xy-th of a plane.
__device__ __forceinline__ void grid_column(const float4* __restrict__ src, Level a, float4* __restrict__ dst, Level b,
                                            int xy, int z0, float sigma_scale) {
    const int y = (int)((unsigned)xy / (unsigned)b.nx), x = xy - y * b.nx;
    int ix, iy;
    float fx, fy;
    lerp_clamped(x, a.nx, b.nx, ix, fx);
    lerp_clamped(y, a.ny, b.ny, iy, fy);
    const int at = iy * a.nx + ix, pitch = a.nx * a.ny;
    const float w00 = (1.0f - fx) * (1.0f - fy), w10 = fx * (1.0f - fy), w01 = (1.0f - fx) * fy, w11 = fx * fy;
    auto plane = [&](int z) {
        const float4* q = src + (z * pitch + at);
        const float4 lo = mix(q[0], w00, q[1], w10), hi = mix(q[a.nx], w01, q[a.nx + 1], w11);
        return make_float4(lo.x + hi.x, lo.y + hi.y, lo.z + hi.z, lo.w + hi.w);
    };
    int have = -2;  // source plane below the pair at hand (the same for every thread of the workgroup)
    float4 p0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), p1 = p0;
    const int zn = min(kColumn, b.nz - z0);
    for (int k = 0; k < zn; ++k) {
        int iz;
        float fz;
        lerp_clamped(z0 + k, a.nz, b.nz, iz, fz);
        if (iz != have) {
            p0 = iz == have + 1 ? p1 : plane(iz);
            p1 = plane(iz + 1);
            have = iz;
        }
        float4 v = mix(p0, 1.0f - fz, p1, fz);
        v.w *= sigma_scale;
        dst[(z0 + k) * (b.nx * b.ny) + xy] = v;
    }
}

// Texel t of all layers.
__device__ __forceinline__ void env_texel(const float4* __restrict__ src, Level a, float4* __restrict__ dst, Level b, int t) {
    const int row = (int)((unsigned)t / (unsigned)b.w), i = t - row * b.w;
    const int l = (int)((unsigned)row / (unsigned)b.h), j = row - l * b.h;
    int i0, i1, j0;
    float fu, fv;
    lerp_periodic(i, a.w, b.w, i0, i1, fu);
    lerp_clamped(j, a.h, b.h, j0, fv);
    const float4* s = src + (l * a.h + j0) * a.w;
    const float4 lo = mix(s[i0], (1.0f - fu) * (1.0f - fv), s[i1], fu * (1.0f - fv));
    const float4 hi = mix(s[a.w + i0], (1.0f - fu) * fv, s[a.w + i1], fu * fv);
    dst[t] = make_float4(lo.x + hi.x, lo.y + hi.y, lo.z + hi.z, lo.w + hi.w);
}

__global__ __launch_bounds__(kBlockUp) void k_upsample(const float4* __restrict__ src, Level a, float4* __restrict__ dst,
                                                      Level b, int layers, int plane_blocks, int grid_blocks,
                                                      float sigma_scale) {
    const int id = blockIdx.x;
    if (id < grid_blocks) {
        const int zc = id / plane_blocks, xy = (id - zc * plane_blocks) * kBlockUp + threadIdx.x;
        if (xy < b.nx * b.ny) grid_column(src, a, dst, b, xy, zc * kColumn, sigma_scale);
    } else {
        const int t = (id - grid_blocks) * kBlockUp + threadIdx.x;
        if (t < layers * b.w * b.h) env_texel(src + a.nx * a.ny * a.nz, a, dst + b.nx * b.ny * b.nz, b, t);
    }
}

}  // namespace

hipError_t launch_upsample(const float* src, int sx, int sy, int sz, int sw, int sh, float* dst, int dx, int dy,
                           int dz, int dw, int dh, int layers, float sigma_scale, hipStream_t st) {
    // (units fit 31 bits: the descriptors are checked)
    const Level a{sx, sy, sz, sw, sh}, b{dx, dy, dz, dw, dh};
    const int plane = (dx * dy + kBlockUp - 1) / kBlockUp;
    const int grid = plane * ((dz + kColumn - 1) / kColumn);
    const int env = layers > 0 ? (layers * dw * dh + kBlockUp - 1) / kBlockUp : 0;
    hipLaunchKernelGGL(k_upsample, dim3((unsigned)(grid + env)), dim3(kBlockUp), 0, st, (const float4*)src, a, (float4*)dst, b,
                       layers, plane, grid, sigma_scale);
    return hipGetLastError();
}

}  // namespace perf
