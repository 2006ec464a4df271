// The feature pass of many small volumes, one launch a pass for all that share a stencil radius (the batched
// launch): the bodies of dvr_features' fixed-radius kernels (features_dev.hpp) with their arguments read from
// a table, so the values are theirs, bit for bit.  A volume is a row of the grid (blockIdx.y); workgroups past
// its last tile end at once.
//
// A kernel node of a HIP graph takes 3-4 us and a volume of 64^3 voxels leaves most of the chip idle, so one pair
// of launches a volume and scale was bound by the launches: the batched launch of 1024 volumes of 16^3 with a
// 32^2 view each 7.68 -> 0.48 ms, 256 of 24^3 with a 64^2 view 1.90 -> 0.40 (quads, two scales 4.97 -> 0.57).
#include "common.hpp"
#include "features_dev.hpp"

namespace dvr {

// The table is addressed through the constant address space, so that the uniform loads of its fields become
// scalar loads; the pointers in it are to global memory (without the cast they would be read as generic ones).
template <typename T>
using CP = const __attribute__((address_space(4))) T *;
template <typename T>
__device__ __forceinline__ T *global_ptr(T *p)
{
    return (T *)(__attribute__((address_space(1))) T *)p;
}

template <int DT, int R>
__global__ __launch_bounds__(256) void k_group_z(uint64_t table)
{
    const auto &it = ((CP<FeatItem>)table)[blockIdx.y];
    const int nx = it.a.nx, ny = it.a.ny, nz = it.a.nz;
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny, per = (plane + 255u) / 256u;
    const uint32_t run = blockIdx.x / per, e = (blockIdx.x - run * per) * 256u + threadIdx.x;
    if (run * kTZ >= (uint32_t)nz || e >= plane) return;
    zpass_run<DT, R, kTZ>(global_ptr(it.a.vol), global_ptr(const_cast<float *>(it.a.ws)), nx, ny, nz, it.taps.ax[2], e,
                          (int)run * kTZ);
}

template <int DT, int LAYOUT, int R>
__global__ __launch_bounds__(NT, (R >= 6 && R <= 9) ? 6 : 1) void k_group_xy(uint64_t table)
{
    using T = XYTileR<R, TX, TY>;
    using S = XYSlab<DT, DT, LAYOUT, R, TX, TY, const __attribute__((address_space(4))) ScaleTaps>;
    __shared__ float F[T::NF > T::NFY ? T::NF : T::NFY];
    const auto &it = ((CP<FeatItem>)table)[blockIdx.y];
    XYArgs a;  // field by field: the table lives in the constant address space
    a.ws = global_ptr(it.a.ws);
    a.vol = global_ptr(it.a.vol);
    a.grad = global_ptr(it.a.grad);
    a.kappa = global_ptr(it.a.kappa);
    a.ves = global_ptr(it.a.ves);
    a.gmax = global_ptr(it.a.gmax);
    a.fro = nullptr;
    a.nx = it.a.nx;
    a.ny = it.a.ny;
    a.nz = it.a.nz;
    for (int k = 0; k < 3; ++k) a.inv2h[k] = it.a.inv2h[k];
    a.c_host = it.a.c_host;
    a.inv2a2 = it.a.inv2a2;
    a.inv2b2 = it.a.inv2b2;
    a.tau = it.a.tau;
    a.first = it.a.first;
    a.fro_pass = 0;
    a.odt = it.a.odt;
    a.layout = it.a.layout;
    const uint32_t tx = (uint32_t)(a.nx + TX - 1) / TX, ty = (uint32_t)(a.ny + TY - 1) / TY;
    const uint32_t z = blockIdx.x / (tx * ty), t = blockIdx.x - z * (tx * ty), row = t / tx;
    if (z >= (uint32_t)a.nz) return;
    S s(a, it.taps, F, F, (int)(t - row * tx) * TX, (int)row * TY);
    s.load((int)z);
    s.store();
    __syncthreads();
    float vmax = s.compute((int)z, s.In, s.Vp);
    if (a.first) {
        vmax = wave_max(vmax);
        if ((threadIdx.x & 63) == 0) atomic_max_pos(a.gmax, vmax);
    }
}

// V quads from the plain V (intensity = false), then the intensity quads over it
template <typename T, typename T4>
__global__ __launch_bounds__(256) void k_group_quads(uint64_t table, bool intensity)
{
    const auto &it = ((CP<FeatItem>)table)[blockIdx.y];
    const uint32_t nx = (uint32_t)it.a.nx, ny = (uint32_t)it.a.ny, nz = (uint32_t)it.a.nz;
    const uint32_t v = blockIdx.x * 256u + threadIdx.x;
    if (v >= nx * ny * nz) return;
    const T *src = (const T *)global_ptr(intensity ? it.a.vol : (const void *)it.a.ves);
    T4 *dst = (T4 *)global_ptr(intensity ? it.a.ves : it.quads);
    quad_of(src, dst, nx, ny, nz, v);
}

template <int R>
static hipError_t group_z(uint64_t table, int n, unsigned groups, int dt, int want, hipStream_t st)
{
    if constexpr (R > kGroupRadius) {
        return hipErrorInvalidValue;
    } else {
        if (want != R) return group_z<R + 1>(table, n, groups, dt, want, st);
        if (dt == DVR_F32) hipLaunchKernelGGL((k_group_z<DVR_F32, R>), dim3(groups, n), dim3(256), 0, st, table);
        else hipLaunchKernelGGL((k_group_z<DVR_F16, R>), dim3(groups, n), dim3(256), 0, st, table);
        return hipGetLastError();
    }
}

template <int R>
static hipError_t group_xy(uint64_t table, int n, unsigned groups, int dt, int layout, int want, hipStream_t st)
{
    if constexpr (R > kGroupRadius) {
        return hipErrorInvalidValue;
    } else {
        if (want != R) return group_xy<R + 1>(table, n, groups, dt, layout, want, st);
        // the instantiations that dvr_features takes for these pairs
#define DVR_GROUP(D, L) hipLaunchKernelGGL((k_group_xy<D, L, R>), dim3(groups, n), dim3(NT), 0, st, table)
        if (dt == DVR_F32 && layout == DVR_PLANAR) DVR_GROUP(DVR_F32, DVR_PLANAR);
        else if (dt == DVR_F32 && layout == DVR_SPLIT) DVR_GROUP(DVR_F32, DVR_SPLIT);
        else if (dt == DVR_F32) DVR_GROUP(DVR_F32, kAnyOut);
        else if (layout == DVR_PLANAR) DVR_GROUP(DVR_F16, DVR_PLANAR);
        else if (layout == DVR_SPLIT) DVR_GROUP(DVR_F16, DVR_SPLIT);
        else DVR_GROUP(DVR_F16, DVR_INTERLEAVED);
#undef DVR_GROUP
        return hipGetLastError();
    }
}

hipError_t launch_group_z(const FeatItem *table, int n, int64_t groups, int dt, int R, hipStream_t st)
{
    return group_z<2>((uint64_t)(uintptr_t)table, n, (unsigned)groups, dt, R, st);
}

hipError_t launch_group_xy(const FeatItem *table, int n, int64_t groups, int dt, int layout, int R, hipStream_t st)
{
    return group_xy<2>((uint64_t)(uintptr_t)table, n, (unsigned)groups, dt, layout, R, st);
}

hipError_t launch_group_quads(const FeatItem *table, int n, int64_t groups, int dt, bool intensity, hipStream_t st)
{
    const uint64_t t = (uint64_t)(uintptr_t)table;
    const dim3 grid((unsigned)groups, (unsigned)n);
    if (dt == DVR_F32) hipLaunchKernelGGL((k_group_quads<uint32_t, uint4>), grid, dim3(256), 0, st, t, intensity);
    else hipLaunchKernelGGL((k_group_quads<uint16_t, ushort4>), grid, dim3(256), 0, st, t, intensity);
    return hipGetLastError();
}

}  // namespace dvr
