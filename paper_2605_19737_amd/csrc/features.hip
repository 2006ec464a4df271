// Feature pass for gfx950: central-difference gradient (Sec. 2.3 Eq. 2), Gaussian-scale Hessian
// (Sec. 1 "multi-scale Hessian analysis"; Sec. 2.3), its eigenvalues, directional curvature
// (Sec. 2.3 Eq. 3) and Frangi vesselness (Sec. 1 "vesselness measures").
//
// The Hessian of the Gaussian-smoothed volume by clamped central differences is a linear
// operator on I; it is applied here as six separable derivative-of-Gaussian filters
//     Hxx = D2x Gy Gz, Hyy = Gx D2y Gz, Hzz = Gx Gy D2z,
//     Hxy = D1x D1y Gz, Hxz = D1x Gy D1z, Hyz = Gx D1y D1z,
// with exact one-sided variants on the first and last voxel of each axis.  Smoothing first and
// differencing afterwards in FP32 cancels away ~1e-5 of the Hessian's range; the combined taps
// keep it at a few 1e-7.
//
// Two kernels per scale:
//   k_zpass_r   a run of 16 slices per lane: (Gz, D1z, D2z) of I along z -> workspace, 12 B/voxel;
//   k_xypass_r  one 64 x 8 (x, y) tile of one z slice per 256-lane workgroup: the three z-filtered
//             fields of the tile plus halo are staged in LDS, the y filters produce six fields
//             (kept in LDS), the x filters give H per voxel, and the epilogue computes the
//             gradient (first scale), |g|_max, k, the eigenvalues of sigma^2 H and V.
// Both take the stencil radius (2..15, every radius there is) as a template parameter; only a volume
// whose in-plane spacings give x and y different radii takes the run-time-radius tile (k_xypass).
#include <math.h>

#include "common.hpp"
#include "features_dev.hpp"

namespace dvr {

// Stencil radii of the fixed-radius kernels: every radius a Gaussian of radius 1 .. DVR_MAX_RADIUS gives.
// At radius 13 (three scales on a 149 x 193 x 224 volume) the tile below takes 0.16 ms a scale where the
// run-time radius of k_xypass took 1.19.
constexpr int kRFastMin = 2, kRFastMax = DVR_MAX_RADIUS + 1;

// z pass (zpass_run): the grid covers each z plane in 256-voxel runs (blockIdx.x, so lanes read
// consecutive x) and the runs of TZ planes (blockIdx.y).
template <int DT, int R, int TZ>
__global__ __launch_bounds__(256) void k_zpass_r(const void *__restrict__ vol, float *__restrict__ ws, int nx, int ny,
                                                 int nz, AxisTaps tz)
{
    const uint32_t e = blockIdx.x * 256u + threadIdx.x;
    if (e >= (uint32_t)nx * (uint32_t)ny) return;
    zpass_run<DT, R, TZ>(vol, ws, nx, ny, nz, tz, e, (int)blockIdx.y * TZ);
}

template <int DT, int R>
static hipError_t launch_z_r(const void *vol, float *ws, const dvr_grid &g, const AxisTaps &tz, hipStream_t st)
{
    if constexpr (R > kRFastMax) {
        return hipErrorInvalidValue;
    } else {
        if (tz.R != R) return launch_z_r<DT, R + 1>(vol, ws, g, tz, st);
        const uint32_t plane = (uint32_t)g.nx * (uint32_t)g.ny;
        dim3 grid((plane + 255) / 256, (g.nz + kTZ - 1) / kTZ);
        hipLaunchKernelGGL((k_zpass_r<DT, R, kTZ>), grid, dim3(256), 0, st, vol, ws, g.nx, g.ny, g.nz, tz);
        return hipGetLastError();
    }
}

template <int DT, int OUT_DT, int LAYOUT>
__global__ __launch_bounds__(NT) void k_xypass(XYArgs a, ScaleTaps taps)
{
    extern __shared__ float lds[];
    float vmax = xy_tile<DT, OUT_DT, LAYOUT, TX, TY>(a, taps, blockIdx.x * TX, blockIdx.y * TY, blockIdx.z, lds);
    if (a.fro_pass || a.first) {
        vmax = wave_max(vmax);
        if ((threadIdx.x & 63) == 0) atomic_max_pos(a.fro_pass ? a.fro : a.gmax, vmax);
    }
}

// Fixed-radius variant (x and y stencil radius R, equal).  One tile of one slice per workgroup, the y-filtered fields written over the staged ones (one LDS area of
// max(NF, NFY) floats): 25 instead of 41 KB at radius 10, six workgroups a CU instead of three.  At
// radii 6-9 the compiler otherwise takes 103-128 VGPRs (four waves per SIMD) for the y filters'
// registers; held to six waves it needs 57-64, without spills (radius 7: 0.142 -> 0.127 ms on the head).
template <int DT, int OUT_DT, int LAYOUT, int R>
__global__ __launch_bounds__(NT, (R >= 6 && R <= 9) ? 6 : 1) void k_xypass_r(XYArgs a, ScaleTaps taps)
{
    using T = XYTileR<R, TX, TY>;
    using S = XYSlab<DT, OUT_DT, LAYOUT, R, TX, TY>;
    __shared__ float F[T::NF > T::NFY ? T::NF : T::NFY];
    S s(a, taps, F, F, blockIdx.x * TX, blockIdx.y * TY);
    const int z = blockIdx.z;
    s.load(z);
    s.store();
    __syncthreads();
    float vmax = s.compute(z, s.In, s.Vp);
    if (a.fro_pass || a.first) {
        vmax = wave_max(vmax);
        if ((threadIdx.x & 63) == 0) atomic_max_pos(a.fro_pass ? a.fro : a.gmax, vmax);
    }
}

template <int DT, int OUT_DT, int LAYOUT, int R>
static hipError_t launch_xy_r(const XYArgs &a, const ScaleTaps &taps, hipStream_t st)
{
    if constexpr (R > kRFastMax) {
        return hipErrorInvalidValue;
    } else {
        if (taps.ax[0].R != R) return launch_xy_r<DT, OUT_DT, LAYOUT, R + 1>(a, taps, st);
        dim3 grid((a.nx + TX - 1) / TX, (a.ny + TY - 1) / TY, a.nz);
        hipLaunchKernelGGL((k_xypass_r<DT, OUT_DT, LAYOUT, R>), grid, dim3(NT), 0, st, a, taps);
        return hipGetLastError();
    }
}

// Brick table: (min, max) of the (DVR_BRICK + 1)^3 voxels of each brick.  Bound by reading the volume
// once, so lanes run along x and a workgroup walks a run of bricks along z, reading every slice once
// (the voxel shared by two bricks of a column included) and each row 5/4 times: 0.19 -> 0.06 ms on a
// 512 x 512 x 400 FP16 volume (210 MB) against one lane per brick that gathers its 125 voxels.
// SRC: 0 F32 volume, 1 F16 volume, 2 F32 records (I at stride 8), 3 F16 records.
// V consecutive voxels of x per lane: 4 (one brick, one vector load a row; rows and base aligned to
// it, which nx % 4 == 0 gives) or 1 (any nx, four lanes a brick).
template <int SRC, int V>
__device__ __forceinline__ void brick_load(const void *__restrict__ src, uint32_t v, float (&f)[V])
{
    if constexpr (V == 4 && SRC == 0) {
        const float4 q = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(src) + v);
        f[0] = q.x; f[1] = q.y; f[2] = q.z; f[3] = q.w;
    } else if constexpr (V == 4) {
        const uint2 q = *reinterpret_cast<const uint2 *>(reinterpret_cast<const __half *>(src) + v);
        const f16x4 h = __builtin_bit_cast(f16x4, q);
        f[0] = (float)h[0]; f[1] = (float)h[1]; f[2] = (float)h[2]; f[3] = (float)h[3];
    } else if constexpr (SRC == 0) f[0] = reinterpret_cast<const float *>(src)[v];
    else if constexpr (SRC == 1) f[0] = __half2float(reinterpret_cast<const __half *>(src)[v]);
    else if constexpr (SRC == 2) f[0] = reinterpret_cast<const float *>(src)[8u * v];
    else f[0] = __half2float(reinterpret_cast<const __half *>(src)[8u * v]);
}

// A wave takes 64 V consecutive voxels of x (blockIdx.x) of brick row by (four to a workgroup) over
// the bricks [run blockIdx.z, ...) of z.
template <int SRC, int V>
__global__ __launch_bounds__(256) void k_bricks(const void *__restrict__ src, float2 *__restrict__ out, int nx, int ny,
                                                int nz, int nbx, int nby, int nbz, int run)
{
    static_assert(DVR_BRICK == 4 && (V == 1 || V == 4), "four voxels a brick along x");
    const int lane = threadIdx.x & 63;
    const int by = (int)(blockIdx.y * 4u + (threadIdx.x >> 6));
    if (by >= nby) return;  // uniform over the wave
    const int xw = (int)blockIdx.x * 64 * V;  // the wave's first voxel
    const int x = xw + lane * V;
    const int xc = min(x, nx - V);  // lanes past the row read its last voxels (their results are not stored)
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    // the voxel after the wave's last one belongs to its last brick too
    const bool tail = lane == 63 && xw + 64 * V < nx;
    const int bz0 = (int)blockIdx.z * run, bz1 = min(bz0 + run, nbz);
    const int y0 = by * DVR_BRICK;
    // min, max over a slice's rows of the lane's voxels, and of the lane's first voxel alone (the last
    // voxel of the brick before)
    float cmn = 0.f, cmx = 0.f, emn = 0.f, emx = 0.f, tmn = 0.f, tmx = 0.f;
    auto slice = [&](int z, float &mn, float &mx, float &fmn, float &fmx, float &lmn, float &lmx) {
        mn = fmn = lmn = INFINITY;
        mx = fmx = lmx = -INFINITY;
#pragma unroll
        for (int r = 0; r <= DVR_BRICK; ++r) {
            const uint32_t row = (uint32_t)z * plane + (uint32_t)min(y0 + r, ny - 1) * (uint32_t)nx;
            float f[V];
            brick_load<SRC, V>(src, row + (uint32_t)xc, f);
            fmn = fminf(fmn, f[0]);
            fmx = fmaxf(fmx, f[0]);
#pragma unroll
            for (int e = 0; e < V; ++e) {
                mn = fminf(mn, f[e]);
                mx = fmaxf(mx, f[e]);
            }
            if (tail) {
                float g[1];
                brick_load<SRC, 1>(src, row + (uint32_t)(xw + 64 * V), g);
                lmn = fminf(lmn, g[0]);
                lmx = fmaxf(lmx, g[0]);
            }
        }
    };
    slice(bz0 * DVR_BRICK, cmn, cmx, emn, emx, tmn, tmx);
    for (int bz = bz0; bz < bz1; ++bz) {
        float mn = cmn, mx = cmx, fmn = emn, fmx = emx, lmn = tmn, lmx = tmx;
#pragma unroll
        for (int k = 1; k <= DVR_BRICK; ++k) {
            slice(min(bz * DVR_BRICK + k, nz - 1), cmn, cmx, emn, emx, tmn, tmx);
            mn = fminf(mn, cmn);
            mx = fmaxf(mx, cmx);
            fmn = fminf(fmn, emn);
            fmx = fmaxf(fmx, emx);
            lmn = fminf(lmn, tmn);
            lmx = fmaxf(lmx, tmx);
        }
        // the brick's fifth column: the first voxel of the next brick's first lane
        int bx;
        float nmn, nmx;
        if constexpr (V == 4) {
            bx = x / DVR_BRICK;
            nmn = __shfl_down(fmn, 1, 64);
            nmx = __shfl_down(fmx, 1, 64);
        } else {
            bx = x / DVR_BRICK;
            mn = fminf(mn, __shfl_xor(mn, 1, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 1, 64));
            mn = fminf(mn, __shfl_xor(mn, 2, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 2, 64));
            nmn = __shfl_down(fmn, 1, 64);  // used by the brick's last lane
            nmx = __shfl_down(fmx, 1, 64);
        }
        if (lane == 63) {
            nmn = lmn;
            nmx = lmx;
        }
        const bool writer = V == 4 || (lane & 3) == 3;
        if (writer && bx < nbx) out[((size_t)bz * nby + by) * nbx + bx] = make_float2(fminf(mn, nmn), fmaxf(mx, nmx));
    }
}

template <int SRC>
static void launch_bricks_t(const void *src, float2 *o, const dvr_grid &g, int nbx, int nby, int nbz, hipStream_t st)
{
    const bool vec = SRC < 2 && g.nx % 4 == 0;
    const unsigned bx = (unsigned)((g.nx + (vec ? 255 : 63)) / (vec ? 256 : 64)), by = (unsigned)((nby + 3) / 4);
    // a run reads 4 run + 1 slices, but only 4096 waves fill the chip: shorter runs on small volumes
    // (a 353 x 74 x 65 one: runs of 4 cost 6 us more than one brick a lane did)
    int run = 4;
    while (run > 1 && (int64_t)bx * nby * ((nbz + run - 1) / run) < 4096) run >>= 1;
    const dim3 grid(bx, by, (unsigned)((nbz + run - 1) / run));
    if (vec)
        hipLaunchKernelGGL((k_bricks<SRC, SRC < 2 ? 4 : 1>), grid, dim3(256), 0, st, src, o, g.nx, g.ny, g.nz, nbx, nby,
                           nbz, run);
    else
        hipLaunchKernelGGL((k_bricks<SRC, 1>), grid, dim3(256), 0, st, src, o, g.nx, g.ny, g.nz, nbx, nby, nbz, run);
}

// One lane per voxel, x fastest: the four rows are read coalesced (mostly from L2), the quad is
// written as one 16- (F32) or 8-byte (F16) store.
template <typename T, typename T4>
__global__ void __launch_bounds__(256) k_quads(const T *__restrict__ src, T4 *__restrict__ dst, uint32_t nx,
                                               uint32_t ny, uint32_t nz)
{
    const uint32_t v = blockIdx.x * 256u + threadIdx.x;
    if (v < nx * ny * nz) quad_of(src, dst, nx, ny, nz, v);
}

hipError_t launch_quads(const void *src, void *dst, const dvr_grid &g, int dtype, hipStream_t st)
{
    const uint32_t n = (uint32_t)g.nx * (uint32_t)g.ny * (uint32_t)g.nz;
    const dim3 grid((n + 255u) / 256u);
    if (dtype == DVR_F32)
        hipLaunchKernelGGL((k_quads<uint32_t, uint4>), grid, dim3(256), 0, st, static_cast<const uint32_t *>(src),
                           static_cast<uint4 *>(dst), (uint32_t)g.nx, (uint32_t)g.ny, (uint32_t)g.nz);
    else
        hipLaunchKernelGGL((k_quads<uint16_t, ushort4>), grid, dim3(256), 0, st, static_cast<const uint16_t *>(src),
                           static_cast<ushort4 *>(dst), (uint32_t)g.nx, (uint32_t)g.ny, (uint32_t)g.nz);
    return hipGetLastError();
}

hipError_t launch_bricks(const void *vol, int vol_dt, const dvr_grid &g, const dvr_features_buf &out, hipStream_t st)
{
    const int nbx = (g.nx - 1 + DVR_BRICK - 1) / DVR_BRICK, nby = (g.ny - 1 + DVR_BRICK - 1) / DVR_BRICK,
              nbz = (g.nz - 1 + DVR_BRICK - 1) / DVR_BRICK;
    float2 *o = reinterpret_cast<float2 *>(out.bricks);
    // the records' I is the volume itself when the dtypes agree (read the contiguous volume then)
    if (out.layout == DVR_INTERLEAVED && out.dtype != vol_dt) {
        if (out.dtype == DVR_F32) launch_bricks_t<2>(out.grad, o, g, nbx, nby, nbz, st);
        else launch_bricks_t<3>(out.grad, o, g, nbx, nby, nbz, st);
    } else if (vol_dt == DVR_F32) {
        launch_bricks_t<0>(vol, o, g, nbx, nby, nbz, st);
    } else {
        launch_bricks_t<1>(vol, o, g, nbx, nby, nbz, st);
    }
    return hipGetLastError();
}

__global__ void k_init_scalars(float *gmax, float *fro)
{
    if (threadIdx.x == 0) {
        if (gmax) *gmax = 0.f;
        if (fro) *fro = 0.f;
    }
}

hipError_t launch_init_scalars(float *gmax, float *ws_scalars, hipStream_t st)
{
    hipLaunchKernelGGL(k_init_scalars, dim3(1), dim3(64), 0, st, gmax, ws_scalars);
    return hipGetLastError();
}

template <int DT, int OUT_DT, int LAYOUT>
static hipError_t launch_xy(const XYArgs &a, const ScaleTaps &taps, hipStream_t st)
{
    const size_t lds = sizeof(float) * xy_lds_floats<TX, TY>(taps.ax[0].R, taps.ax[1].R);
    dim3 grid((a.nx + TX - 1) / TX, (a.ny + TY - 1) / TY, a.nz);
    hipLaunchKernelGGL((k_xypass<DT, OUT_DT, LAYOUT>), grid, dim3(NT), lds, st, a, taps);
    return hipGetLastError();
}

static hipError_t launch_z(const void *vol, int vol_dt, const dvr_grid &g, const AxisTaps &tz, float *ws_fields,
                           hipStream_t st)
{
    return (vol_dt == DVR_F32) ? launch_z_r<DVR_F32, kRFastMin>(vol, ws_fields, g, tz, st)
                               : launch_z_r<DVR_F16, kRFastMin>(vol, ws_fields, g, tz, st);
}

hipError_t launch_hessian(const void *vol, int vol_dt, const dvr_grid &g, const ScaleTaps &taps, float *ws_fields,
                          float *H, hipStream_t st)
{
    hipError_t e = launch_z(vol, vol_dt, g, taps.ax[2], ws_fields, st);
    if (e != hipSuccess) return e;
    XYArgs a = {};
    a.ws = ws_fields;
    a.vol = vol;
    a.grad = H;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.first = 0;
    a.fro_pass = 0;
    const int R = taps.ax[0].R;
    if (R == taps.ax[1].R)
        return (vol_dt == DVR_F32) ? launch_xy_r<DVR_F32, DVR_F32, kHessianOut, kRFastMin>(a, taps, st)
                                   : launch_xy_r<DVR_F16, DVR_F32, kHessianOut, kRFastMin>(a, taps, st);
    if (vol_dt == DVR_F32) return launch_xy<DVR_F32, DVR_F32, kHessianOut>(a, taps, st);
    return launch_xy<DVR_F16, DVR_F32, kHessianOut>(a, taps, st);
}

hipError_t launch_features_scale(const void *vol, int vol_dt, const dvr_grid &g, const ScaleTaps &taps,
                                 int scale_index, bool last_scale, const dvr_feature_params &fp,
                                 const dvr_features_buf &out, float *ws_fields, float *ws_scalars,
                                 bool fro_pass, hipStream_t st)
{
    (void)last_scale;
    hipError_t e = launch_z(vol, vol_dt, g, taps.ax[2], ws_fields, st);
    if (e != hipSuccess) return e;

    const XYArgs a = xy_args(vol, g, fp, out, ws_fields, ws_scalars, scale_index, fro_pass);
    const int odt = out.dtype, lay = out.layout;
    if (taps.ax[0].R == taps.ax[1].R) {
        // the layouts that are rendered most have kernels of their own; the others share one whose
        // storage type and layout are run-time values (2-11 % slower than its own kernel where both
        // exist, 1.4-1.8x faster per call than the run-time-radius tile they took before)
        if (vol_dt == DVR_F32 && odt == DVR_F32 && lay == DVR_PLANAR)
            return launch_xy_r<DVR_F32, DVR_F32, DVR_PLANAR, kRFastMin>(a, taps, st);
        if (vol_dt == DVR_F16 && odt == DVR_F16 && lay == DVR_INTERLEAVED)
            return launch_xy_r<DVR_F16, DVR_F16, DVR_INTERLEAVED, kRFastMin>(a, taps, st);
        if (vol_dt == DVR_F32 && odt == DVR_F32 && lay == DVR_SPLIT)
            return launch_xy_r<DVR_F32, DVR_F32, DVR_SPLIT, kRFastMin>(a, taps, st);
        if (vol_dt == DVR_F16 && odt == DVR_F16 && lay == DVR_SPLIT)
            return launch_xy_r<DVR_F16, DVR_F16, DVR_SPLIT, kRFastMin>(a, taps, st);
        if (vol_dt == DVR_F16 && odt == DVR_F16 && lay == DVR_PLANAR)  // the split layout's values, bit for bit
            return launch_xy_r<DVR_F16, DVR_F16, DVR_PLANAR, kRFastMin>(a, taps, st);
        return (vol_dt == DVR_F32) ? launch_xy_r<DVR_F32, DVR_F32, kAnyOut, kRFastMin>(a, taps, st)
                                   : launch_xy_r<DVR_F16, DVR_F32, kAnyOut, kRFastMin>(a, taps, st);
    }
    // in-plane spacings so unequal that the radii differ: the run-time-radius tile
#define DVR_XY(D, O, L) \
    if (vol_dt == D && odt == O && lay == L) return launch_xy<D, O, L>(a, taps, st);
    DVR_XY(DVR_F32, DVR_F32, DVR_PLANAR)
    DVR_XY(DVR_F32, DVR_F32, DVR_INTERLEAVED)
    DVR_XY(DVR_F32, DVR_F16, DVR_PLANAR)
    DVR_XY(DVR_F32, DVR_F16, DVR_INTERLEAVED)
    DVR_XY(DVR_F16, DVR_F32, DVR_PLANAR)
    DVR_XY(DVR_F16, DVR_F32, DVR_INTERLEAVED)
    DVR_XY(DVR_F16, DVR_F16, DVR_PLANAR)
    DVR_XY(DVR_F16, DVR_F16, DVR_INTERLEAVED)
    DVR_XY(DVR_F32, DVR_F32, DVR_SPLIT)
    DVR_XY(DVR_F32, DVR_F16, DVR_SPLIT)
    DVR_XY(DVR_F16, DVR_F32, DVR_SPLIT)
    DVR_XY(DVR_F16, DVR_F16, DVR_SPLIT)
#undef DVR_XY
    return hipErrorInvalidValue;
}

}  // namespace dvr
