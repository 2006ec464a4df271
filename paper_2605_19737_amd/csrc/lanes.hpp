// The split of a launch's rays over lanes and workgroups, shared by the per-call raymarch (render.hip) and
// the batched launch (batch.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "render_args.hpp"

namespace dvr {

// Host: how a view samples the volume.
struct ViewGeo {
    double pitch;  // pixel pitch in voxels, the larger of a pixel's two steps
    double chord;  // samples of a mean ray through the box
    double hit;    // share of the pixels whose ray meets the box, at most
};

// (at the box centre for a perspective view; a box partly outside the image is counted whole)
inline ViewGeo view_geo(const KCam &cam, int W, int H, const KGrid &g)
{
    double scale = 1.0, du = 0.0, dv = 0.0, d[3], ext[3], dist = 0.0, dir = 0.0;
    for (int a = 0; a < 3; ++a) {
        ext[a] = (g.n[a] - 1) * (double)g.h[a];
        const double to = 0.5 * ext[a] - cam.o[a];
        d[a] = cam.d0[a];
        if (cam.persp) d[a] += 0.5 * W * (double)cam.du[a] + 0.5 * H * (double)cam.dv[a];
        dist += to * to;
        dir += d[a] * d[a];
        du += (cam.du[a] / (double)g.h[a]) * (cam.du[a] / (double)g.h[a]);
        dv += (cam.dv[a] / (double)g.h[a]) * (cam.dv[a] / (double)g.h[a]);
    }
    if (cam.persp && dir > 0.0) scale = sqrt(dist / dir);
    ViewGeo v;
    v.pitch = scale * sqrt(du > dv ? du : dv);
    // the box's shadow along the view, and a pixel's area, in mm^2
    const double area = (fabs(d[0]) * ext[1] * ext[2] + fabs(d[1]) * ext[0] * ext[2] + fabs(d[2]) * ext[0] * ext[1]) /
                        (dir > 0.0 ? sqrt(dir) : 1.0);
    double px = 0.0;
    for (int a = 0; a < 3; ++a) {
        const int b = (a + 1) % 3, c = (a + 2) % 3;
        const double x = (double)cam.du[b] * cam.dv[c] - (double)cam.du[c] * cam.dv[b];
        px += x * x;
    }
    px = scale * scale * sqrt(px);
    v.chord = area > 0.0 ? ext[0] * ext[1] * ext[2] / (area * (double)g.delta_hi) : 0.0;
    v.hit = px > 0.0 && area < px * W * H ? area / (px * W * H) : 1.0;
    return v;
}

// Side in pixels of a workgroup's tile with G lanes per ray.
__host__ __device__ constexpr uint32_t tile_side(int G) { return G == 1 ? 16 : (G == 4 ? 8 : 4); }

// Workgroups that a launch of 256 threads each may have: HIP refuses gridDim.x * blockDim.x >= 2^32.
constexpr uint64_t kMaxGroups = (1u << 24) - 1;

// Host: workgroups of ncam W x H views with G lanes per ray, rounded up to the 8 XCDs: one a tile, or
// (spread) four a block of 2 x 2 tiles.
inline uint64_t tile_groups(int W, int H, int ncam, int G, uint32_t spread)
{
    const uint64_t side = (uint64_t)tile_side(G) * (spread ? 2u : 1u);
    const uint64_t n = (((uint64_t)W + side - 1u) / side) * (((uint64_t)H + side - 1u) / side) * (uint64_t)ncam;
    return (n + 7u) / 8u * (spread ? 32u : 8u);
}

struct RaySplit {
    int lanes;           // per ray
    uint32_t spread;     // the XCDs take blocks of 2 x 2 tiles in turn (KLaunch::spread)
    uint32_t parts = 1;  // adjoint: workgroups that share a tile's blocks of rays
};

// Host: the split s with fewer lanes per ray, then with the XCDs' contiguous tiles, as far as the launch
// needs it to fit in one grid (more than 2^30 pixels with 4 lanes; images of a few columns or rows, where
// blocks of 2 x 2 tiles are mostly padding).  The adjoint's grid is that of one lane per ray.
inline RaySplit fit_split(RaySplit s, int W, int H, int ncam, bool adjoint)
{
    while (!adjoint && s.lanes > 1 && tile_groups(W, H, ncam, s.lanes, s.spread) > kMaxGroups) s.lanes /= 4;
    if (tile_groups(W, H, ncam, adjoint ? 1 : s.lanes, s.spread) > kMaxGroups) s.spread = 0;
    return s;
}

// Host: lanes per ray of the forward raymarch, by the rays of the launch and the pitch. Few rays: with
// one lane a ray the chip needs a million rays to hide a ray's chain of dependent samples and to even
// out the rays' lengths. One view of a 64^3 volume in the quad layout, 1 / 4 / 16 lanes: 128^2 214 / 66
// / 66 us, 256^2 201 / 121 / 120, 512^2 393 / 231 / 365; of a head: 398 / 128 / 96, 386 / 182 / 187,
// 529 / 268 / 568, 1024^2 552 / 437 (four such views: 1014 / 989 at 768^2, eight 2654 / 3236 at
// 1024^2). 16 lanes hold a wave's samples closer together, which pays longer where a sample touches
// more cache lines: FP32 (64^3 at 256^2, split 174 us with 4 lanes, 134 with 16; FP16 interleaved 108,
// 128) and above all FP32 planes (267, 155; 384^2 328, 299). Coarse views: 8 x 8 rays spread over many
// cache lines; a 152 x 229 x 177 volume at 512^2 x 32 (1.35 voxels a pixel) 10.8 ms with one lane, 7.4
// with 4, at 180^2 x 20 (3.8) 3.6, 2.05 and with 16 1.19; a 512 x 512 x 400 one at 1024^2 x 2 (0.8)
// 3.1, 2.4.
//
// More lanes repeat the ray set-up and the workgroup's transfer function for every pixel, also where the ray
// misses: three more lanes cost 33 ns a thousand rays (50 with more than 16 knots), 15 four times as much.
// What they save is the chain of a mean ray's samples (1 us each; 0.25 from 4 lanes to 16) and, on coarse
// views, 0.5 ps a sample (4 from 4 lanes to 16), so a volume that is thin or small in its image keeps fewer.
// us, 1 / 4 / 16 lanes: 231 x 286 x 6 (27 samples) in three 700 x 500 views 75 / 93 / 294 over a ninth of the
// image, 75 / 70 / 234 at 4.7 voxels a pixel, in three 1500^2 views at 1.5 131 / 328 / 1290; a head (257) in
// two 1024^2 views over a 70th 554 / 258 / 476, in nine 2048^2 ones 1695 / 2327 / 8289.
inline int fwd_lanes(double rays, int layout, int dtype, int K, const ViewGeo &v)
{
    const double most16 = dtype == DVR_F16 ? 40960 : (layout == DVR_PLANAR ? 163840 : 81920);
    const double setup = (K > 16 ? 5e-5 : 3.3e-5) * rays, samples = v.chord * v.hit * rays;
    if (rays <= most16) return 16;
    if (v.pitch > 2.5 && rays <= 1200000 && 0.25 * v.chord + 4e-6 * samples > 4.0 * setup) return 16;
    if (rays > 1200000 && v.pitch <= 0.6) return 1;
    return v.chord + 5e-7 * samples > setup ? 4 : 1;
}

}  // namespace dvr
