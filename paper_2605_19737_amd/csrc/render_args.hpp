// Kernel-argument records of the raymarcher (passed by value; no device-side parameter buffers,
// so a launch records into a HIP graph with nothing else to copy).
#pragma once

#include <math.h>
#include <stdint.h>

#include "dvr.h"

namespace dvr {

constexpr int kCamChunk = 32;  // cameras per launch (kernel arguments stay under 4 KB)

struct KCam {
    int32_t persp;
    float o[3], d0[3], du[3], dv[3];
};

struct KFeat {
    const void *vol;  // planar: the intensity volume (same dtype as the features)
    const void *grad, *kappa, *ves;
    const float *gmax;
    int32_t dtype, layout;
    const float *bricks;  // [nb2][nb1][nb0][2] intensity (min, max) per brick, or null (no skipping)
    int32_t nb[3];
};

struct KGrid {
    int32_t n[3];
    float h[3];
    float delta_hi, delta_lo;    // step_vox * min(h) in mm, exactly: the sum of the two (the product of
                                 // two FP32 numbers has at most 48 significant bits)
    float ih_hi[3], ih_lo[3];    // 1 / h as a double-float pair (~48 bits)
    float idelta_hi, idelta_lo;  // 1 / (step_vox * min(h)) likewise
};

struct KTF {
    int32_t K;
    const float *knots, *rgba;
};

struct KRender {
    float lg, omlg, lk, omlk, k0, lv;
    float Tstop;  // stop once T <= Tstop (1 - et_alpha, or 2^-24 without early termination)
};

struct KLaunch {
    int32_t W, H, ncam, cam_base;
    uint32_t spread;        // the XCDs take the launch's blocks of tiles in turn (else whole views)
    float *out;             // [cam][H][W][4]
    float *T_last;          // [cam][H][W] or null
    int32_t *k_last;        // [cam][H][W] or null
    const float *dout;      // backward: dL/d rgba
    float *dtf;             // backward: dL/d TF values [K][4]
    float *dvol;            // backward: dL/d I [N] or null
    float *dfeat = nullptr;  // backward with feature gradients: dL/d(gx, gy, gz, k, V) as [5][N], or null
    float *dgmax = nullptr;  // backward with feature gradients: dL/d gmax [1]
    unsigned long long *counters;  // forward: evaluated samples, shaded samples (or null)
    KCam cams[kCamChunk];
};

struct RenderArgs {
    KFeat feat;
    KGrid grid;
    KTF tf;
    KRender rp;
    KLaunch launch;  // template: cams filled per chunk
    const KCam *cams;
    int32_t ncam;
};

// Host: a double as the pair hi + lo of FP32 numbers (exact for the 48-bit product step_vox * hmin).
inline void split2(double v, float &hi, float &lo)
{
    hi = (float)v;
    lo = (float)(v - (double)hi);
}

// the grid's spacing and segment-length fields of KGrid, from the FP32 spacings and step
inline void set_grid_steps(KGrid &g, const float h[3], float step_vox)
{
    float hmin = h[0];
    if (h[1] < hmin) hmin = h[1];
    if (h[2] < hmin) hmin = h[2];
    const double d = (double)step_vox * (double)hmin;
    split2(d, g.delta_hi, g.delta_lo);
    split2(1.0 / d, g.idelta_hi, g.idelta_lo);
    for (int a = 0; a < 3; ++a) {
        g.h[a] = h[a];
        split2(1.0 / (double)h[a], g.ih_hi[a], g.ih_lo[a]);
    }
}

// Host: pixel pitch of a view in voxels, the larger of a pixel's two steps (at the box centre for a
// perspective view).
inline double pixel_pitch(const KCam &cam, int W, int H, const KGrid &g)
{
    double scale = 1.0, du = 0.0, dv = 0.0;
    if (cam.persp) {
        double dist = 0.0, dir = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double to = 0.5 * (g.n[a] - 1) * (double)g.h[a] - cam.o[a];
            const double d = cam.d0[a] + 0.5 * W * (double)cam.du[a] + 0.5 * H * (double)cam.dv[a];
            dist += to * to;
            dir += d * d;
        }
        scale = dir > 0.0 ? sqrt(dist / dir) : 1.0;
    }
    for (int a = 0; a < 3; ++a) {
        du += (cam.du[a] / (double)g.h[a]) * (cam.du[a] / (double)g.h[a]);
        dv += (cam.dv[a] / (double)g.h[a]) * (cam.dv[a] / (double)g.h[a]);
    }
    return scale * sqrt(du > dv ? du : dv);
}

// Side in pixels of a workgroup's tile with G lanes per ray.
__host__ __device__ constexpr uint32_t tile_side(int G) { return G == 1 ? 16 : (G == 4 ? 8 : 4); }

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
inline int fwd_lanes(double rays, int layout, int dtype, double pitch)
{
    const double most16 = dtype == DVR_F16 ? 40960 : (layout == DVR_PLANAR ? 163840 : 81920);
    if (rays <= most16 || (pitch > 2.5 && rays <= 1200000)) return 16;
    return rays <= 1200000 || pitch > 0.6 ? 4 : 1;
}

}  // namespace dvr
