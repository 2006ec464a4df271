// Batched launch: the feature pass of many volumes and the raymarch of many views, recorded once in a HIP
// graph.
//
//   k_batch_init   clears the stage word, the error flag and every volume's |g|_max;
//   the feature pass of every volume with the kernels of dvr_features (features.hip), small volumes in
//     shared launches (features_group.hip), on up to kLanes parallel branches of the graph, each with a
//     workspace of its own;
//   k_batch_mark   sets the stage word once every branch is done;
//   k_batch_rays   the tiles of every view: one workgroup a tile, each taking its view and tile from a
//     table of blocks of 2 x 2 tiles, each view's dealt to the XCDs in turn; one launch for each number
//     of lanes per ray (1, 4, 16) that the views take.
//
// Bound by the rays' gathers (texture data busy on 99 % of the cycles, VALU issue 82 %; features 0.7 of 6.7 ms
// on eight thick-slice volumes of 2.2-6.1 M voxels with four 512^2 views each, split FP32).  One persistent
// kernel that drained a queue of feature and ray items took 10.5 ms there: the feature items' 168 VGPRs held
// the rays to three waves a SIMD, neighbouring tiles went to different XCDs, and every feature item wrote the
// L2 back.  The tile table in blocks of 1 / 2 x 2 / 4 x 4 / 8 x 8 tiles: 11.0 / 6.69 / 6.75 / 6.98 ms; 1 / 2 / 4
// feature branches: 6.86 / 6.75 / 6.69.  64 such volumes, tuned, 69 -> 62 ms; one to four views of two volumes
// of 1-3 M voxels 3.3-4.1 times faster.
//
// A ray tile checks that the stage word says the features are there, and sets the error flag instead of
// hanging.  The graph orders the mark before the rays, so the check is one load that finds it set: it waits, and
// DVR_E_TIMEOUT is reported, only under the test variable DVR_BATCH_TEST_TIMEOUT.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <fstream>
#include <map>
#include <memory>
#include <sstream>
#include <string>
#include <vector>

#include "common.hpp"
#include "features_dev.hpp"
#include "host.hpp"
#include "lanes.hpp"
#include "render_args.hpp"
#include "render_dev.hpp"

namespace dvr {

constexpr unsigned kMaxSpin = 1u << 23;  // polls of ~0.5 us: a wait gives up after several seconds
constexpr int kMaxVolScale = 8192;       // volumes x scales per plan
constexpr int kLanes = 4;                // feature branches of the graph (the hardware queues of a process)

struct BBlock {      // 2 x 2 tiles
    int32_t view;    // -1: none (padding)
    int32_t tx, ty;  // its first tile
    int32_t pad;
};

struct BView {
    KCam cam;
    KFeat feat;
    KGrid grid;
    int32_t W, H;
    unsigned need;  // the stage the view waits for
    float *rgba;
    float *T_last;
    int32_t *k_last;
};

// Read-only tables are addressed through the constant address space so that the uniform loads
// of their fields become scalar loads (held in SGPRs) rather than per-lane vector loads.
template <typename T>
using CP = const __attribute__((address_space(4))) T *;

struct RayArgs {
    uint64_t blocks;  // BBlock[gridDim.x / 4]
    uint64_t views;  // BView[nview]
    unsigned *stage, *err;
    unsigned max_spin;  // bound of the wait (polls)
    int32_t ray_tile;
    KTF tf;
    KRender rp;
};

// Thread 0: wait until *stage >= need (bounded).
__device__ __forceinline__ void wait_for(unsigned *stage, unsigned need, unsigned *err, unsigned max_spin)
{
    if (threadIdx.x != 0) return;
    unsigned n = 0;
    while (__hip_atomic_load(stage, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
        if (++n > max_spin) {
            atomicOr(err, 1u);
            break;
        }
        __builtin_amdgcn_s_sleep(8);
    }
}

// pixel of this lane's ray in tile (tx, ty); with one lane per ray ray_tile gives the rays of a wave
template <int G>
__device__ __forceinline__ void ray_pixel(int ray_tile, int tx, int ty, int &pi, int &pj)
{
    constexpr int S = (int)tile_side(G);
    const int lane = (int)(threadIdx.x & 63u) / G, wv = threadIdx.x >> 6;
    int ox, oy;
    if (G == 1 && ray_tile == 1) {         // 16 x 4 per wave, waves stacked in y
        ox = lane & 15;
        oy = wv * 4 + (lane >> 4);
    } else if (G == 1 && ray_tile == 2) {  // 4 x 16 per wave, waves side by side in x
        ox = wv * 4 + (lane & 3);
        oy = lane >> 2;
    } else {                               // square, 2 x 2 waves
        ox = (wv & 1) * (S / 2) + lane % (S / 2);
        oy = (wv >> 1) * (S / 2) + lane / (S / 2);
    }
    pi = tx * S + ox;
    pj = ty * S + oy;
}

// One tile of one view per workgroup, G lanes per ray: k_render with the view's records read from the
// tables.  Bound like it, by gathers and instruction issue.
template <int LAYOUT, int DT, int KMAX, int G>
__global__ __launch_bounds__(256, (LAYOUT == DVR_QUAD && DT == DVR_F16 && G == 1) ? 5 : 1) void k_batch_rays(RayArgs A)
{
    // workgroup b runs on XCD b % 8; the four tiles of a block are neighbours there
    const auto &B = ((CP<BBlock>)A.blocks)[(blockIdx.x >> 5) * 8u + (blockIdx.x & 7u)];
    const int view = B.view;
    if (view < 0) return;
    __shared__ TFShared<KMAX> sh;
    float kx[KMAX];
    tf_load<KMAX>(sh, kx, A.tf);
    const auto &V = ((CP<BView>)A.views)[view];
    wait_for(A.stage, V.need, A.err, A.max_spin);
    __syncthreads();
    KFeat f;  // field by field: V lives in the constant address space
    f.vol = V.feat.vol;
    f.grad = V.feat.grad;
    f.kappa = V.feat.kappa;
    f.ves = V.feat.ves;
    f.gmax = V.feat.gmax;
    f.dtype = DT;
    f.layout = LAYOUT;
    f.bricks = nullptr;  // the batched launch builds no brick tables
    f.nb[0] = f.nb[1] = f.nb[2] = 0;
    KGrid g;
    KCam cam;
    cam.persp = V.cam.persp;
    for (int k = 0; k < 3; ++k) {
        g.n[k] = V.grid.n[k];
        g.h[k] = V.grid.h[k];
        g.ih_hi[k] = V.grid.ih_hi[k];
        g.ih_lo[k] = V.grid.ih_lo[k];
        cam.o[k] = V.cam.o[k];
        cam.d0[k] = V.cam.d0[k];
        cam.du[k] = V.cam.du[k];
        cam.dv[k] = V.cam.dv[k];
    }
    g.delta_hi = V.grid.delta_hi;
    g.delta_lo = V.grid.delta_lo;
    g.idelta_hi = V.grid.idelta_hi;
    g.idelta_lo = V.grid.idelta_lo;
    const float gm = *f.gmax;
    const float invg = gm > 0.f ? 1.f / gm : 0.f;
    int pi, pj;
    const int e = (int)(blockIdx.x >> 3) & 3;
    ray_pixel<G>(A.ray_tile, B.tx + (e & 1), B.ty + (e >> 1), pi, pj);
    const bool valid = pi < V.W && pj < V.H;
    RayGeo r;
    r.N = 0;
    if (valid) r = ray_setup(cam, pi, pj, g);
    RayOut o;
    if constexpr (G == 1) o = march_fwd<LAYOUT, DT, KMAX>(f, g, sh, kx, A.rp, invg, r);
    else o = march_fwd_group<LAYOUT, DT, KMAX, G>(f, g, sh, kx, A.rp, invg, r);
    if (valid && (threadIdx.x & (G - 1)) == 0) {
        const size_t pix = (size_t)pj * V.W + pi;
        reinterpret_cast<float4 *>(V.rgba)[pix] = make_float4(o.C0, o.C1, o.C2, o.A);
        if (V.T_last) {
            V.T_last[pix] = o.Tprev;
            if (V.k_last) V.k_last[pix] = o.last;
        }
    }
}

// Clear the stage word, the error flag and every volume's |g|_max (no memset nodes in the graph).
__global__ void k_batch_init(unsigned *stage, unsigned *err, float *const *gmax, int nvol)
{
    if (threadIdx.x == 0) {
        *stage = 0u;
        *err = 0u;
    }
    for (int v = threadIdx.x; v < nvol; v += blockDim.x) *gmax[v] = 0.f;
}

__global__ void k_batch_mark(unsigned *stage)
{
    if (threadIdx.x == 0) *stage = 1u;
}

// ------------------------------------------------------------------------------------------------
// host side

template <int LAYOUT, int DT, int KMAX>
static hipError_t launch_rays_k(const RayArgs &A, int lanes, unsigned grid, hipStream_t st)
{
    if (lanes == 16) hipLaunchKernelGGL((k_batch_rays<LAYOUT, DT, KMAX, 16>), dim3(grid), dim3(256), 0, st, A);
    else if (lanes == 4) hipLaunchKernelGGL((k_batch_rays<LAYOUT, DT, KMAX, 4>), dim3(grid), dim3(256), 0, st, A);
    else hipLaunchKernelGGL((k_batch_rays<LAYOUT, DT, KMAX, 1>), dim3(grid), dim3(256), 0, st, A);
    return hipGetLastError();
}

static hipError_t launch_rays(const RayArgs &A, int layout, int dt, int lanes, unsigned grid, hipStream_t st)
{
#define DVR_R(L, D)                                                                \
    if (layout == L && dt == D) {                                                  \
        if (A.tf.K <= 8) return launch_rays_k<L, D, 8>(A, lanes, grid, st);        \
        if (A.tf.K <= 16) return launch_rays_k<L, D, 16>(A, lanes, grid, st);      \
        return launch_rays_k<L, D, 64>(A, lanes, grid, st);                        \
    }
    DVR_R(DVR_PLANAR, DVR_F32)
    DVR_R(DVR_PLANAR, DVR_F16)
    DVR_R(DVR_INTERLEAVED, DVR_F32)
    DVR_R(DVR_INTERLEAVED, DVR_F16)
    DVR_R(DVR_SPLIT, DVR_F32)
    DVR_R(DVR_SPLIT, DVR_F16)
    DVR_R(DVR_QUAD, DVR_F32)
    DVR_R(DVR_QUAD, DVR_F16)
#undef DVR_R
    return hipErrorInvalidValue;
}

}  // namespace dvr

using namespace dvr;
using namespace dvr::host;

struct dvr_batch {
    hipStream_t stream = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    char *mem = nullptr;  // tables, stage word, workspaces
    unsigned *d_err = nullptr;
    dvr_tune tune;
};

// appends the nodes that the next one recorded on the capturing stream would follow
static hipError_t capture_tail(hipStream_t st, std::vector<hipGraphNode_t> &nodes)
{
    hipStreamCaptureStatus status;
    const hipGraphNode_t *deps = nullptr;
    size_t n = 0;
    const hipError_t e = hipStreamGetCaptureInfo_v2(st, &status, nullptr, nullptr, &deps, &n);
    if (e != hipSuccess) return e;
    if (status != hipStreamCaptureStatusActive || n == 0) return hipErrorStreamCaptureInvalidated;
    nodes.insert(nodes.end(), deps, deps + n);
    return hipSuccess;
}

// ------------------------------------------------------------------------------------------------
// small volumes in shared launches

constexpr int64_t kGroupVox = 1 << 20;   // a volume up to which it shares launches
constexpr int64_t kGroupSum = 4 << 20;   // voxels of a group: bounds its workspace (50 MB)

struct Unit {  // of the feature pass: one volume, or a group
    int64_t vox;
    std::vector<int> vols;
    bool shared = false;  // the kernels of features_group.hip
    int lane = 0;
};

enum { kRunZ = 0, kRunXY = 1, kRunQuadV = 2, kRunQuadI = 3 };
struct GroupRun {  // one launch of a group
    int unit, kind, R;
    int64_t groups;  // workgroups of its largest volume
    size_t first;    // table rows
    int count;
};

// Volumes whose launches can be shared: small ones whose stencil radii the shared kernels have.  The features
// of a batch, us, launches of their own / shared in groups of 4 M / 16 M / 64 M voxels (FP32 split, one scale;
// FP16 quads, two): 4 x 32^3 73 / 32 / 32 / 32, 120 / 53 / 53 / 53; 64 x 64^3 672 / 325 / 358 / 350, 1468 / 705 /
// 750 / 753; 32 x 96^3 686 / 584 / 609 / 632, 1399 / 1232 / 1284 / 1408; 16 x 128^3 564 / 571 / 570 / 599, 1199 /
// 1239 / 1287 / 1340.
// A volume of more slices, or rows of tiles, than a grid has workgroups along an axis takes the shared kernels
// whatever its size: their grid runs along x alone.
static bool too_tall(const dvr_grid &g)
{
    return (unsigned)g.nz > kMaxGridYZ || (unsigned)(g.ny + TY - 1) / TY > kMaxGridYZ;
}

static bool groupable(const dvr_grid &g, const dvr_feature_params &fp)
{
    if (nvox(&g) > kGroupVox && !too_tall(g)) return false;
    for (int sc = 0; sc < fp.nsigma; ++sc) {
        const double sg = fp.sigma_mm[sc];
        const int rx = gauss_radius(sg / g.hx) + 1, ry = gauss_radius(sg / g.hy) + 1, rz = gauss_radius(sg / g.hz) + 1;
        if (rx != ry || rx > kGroupRadius || rz > kGroupRadius) return false;
    }
    return true;
}

// The launches of unit u (its workspace taken to start at address 0), their table rows appended to items: for
// each scale the z passes, one a radius, then the x-y passes; the quads after the last scale.
static void group_runs(const dvr_batch_desc &d, const std::vector<dvr_features_buf> &feats, int u, const Unit &unit,
                       std::vector<FeatItem> &items, std::vector<GroupRun> &runs)
{
    const dvr_feature_params &fp = d.fp;
    const bool quad = feats[unit.vols[0]].layout == DVR_QUAD;
    for (int sc = 0; sc < fp.nsigma; ++sc) {
        std::vector<FeatItem> rows;
        size_t off = 0;
        for (int v : unit.vols) {
            const dvr_grid &g = d.vols[v].grid;
            dvr_features_buf out = feats[v];
            FeatItem it;
            it.quads = out.ves;
            if (quad) {
                out.layout = DVR_SPLIT;
                out.ves = out.iquad;
            }
            it.a = xy_args(d.vols[v].vol, g, fp, out, (const float *)(uintptr_t)(4 * off), nullptr, sc, false);
            const double sg = fp.sigma_mm[sc], h[3] = {g.hx, g.hy, g.hz};
            for (int a = 0; a < 3; ++a) axis_taps(sg / h[a], h[a], it.taps.ax[a]);
            it.taps.sigma2 = (float)(sg * sg);
            rows.push_back(it);
            off += 3 * (size_t)nvox(&g);
        }
        // one launch for the rows of a radius whose workgroups are within a factor of four: the others of a
        // row end at once, but are launched
        auto add = [&](int kind, int axis) {
            std::vector<std::pair<int64_t, size_t>> by_size;
            for (size_t i = 0; i < rows.size(); ++i) {
                const int64_t nx = rows[i].a.nx, ny = rows[i].a.ny, nz = rows[i].a.nz;
                by_size.push_back({kind == kRunZ    ? (nx * ny + 255) / 256 * ((nz + kTZ - 1) / kTZ)
                                   : kind == kRunXY ? (nx + TX - 1) / TX * ((ny + TY - 1) / TY) * nz
                                                    : (nx * ny * nz + 255) / 256,
                                   i});
            }
            std::sort(by_size.rbegin(), by_size.rend());
            const int lo = axis < 0 ? 0 : 2, hi = axis < 0 ? 0 : kGroupRadius;
            for (int R = lo; R <= hi; ++R) {
                GroupRun run = {u, kind, R, 0, 0, 0};
                for (const auto &[n, i] : by_size) {
                    if (axis >= 0 && rows[i].taps.ax[axis].R != R) continue;
                    if (run.count && n * 4 < run.groups) {
                        runs.push_back(run);
                        run.count = 0;
                    }
                    if (!run.count) {
                        run.groups = n;
                        run.first = items.size();
                    }
                    items.push_back(rows[i]);
                    ++run.count;
                }
                if (run.count) runs.push_back(run);
            }
        };
        add(kRunZ, 2);
        add(kRunXY, 0);
        if (quad && sc == fp.nsigma - 1) {
            add(kRunQuadV, -1);
            add(kRunQuadI, -1);
        }
    }
}

static hipError_t launch_run(const GroupRun &g, const FeatItem *table, int dt, int layout, hipStream_t st)
{
    const FeatItem *t = table + g.first;
    if (g.kind == kRunZ) return launch_group_z(t, g.count, g.groups, dt, g.R, st);
    if (g.kind == kRunXY) return launch_group_xy(t, g.count, g.groups, dt, layout == DVR_QUAD ? DVR_SPLIT : layout, g.R, st);
    return launch_group_quads(t, g.count, g.groups, dt, g.kind == kRunQuadI, st);
}

static void plan_free(dvr_batch *p)
{
    if (!p) return;
    if (p->exec) hipGraphExecDestroy(p->exec);
    if (p->graph) hipGraphDestroy(p->graph);
    if (p->stream) hipStreamDestroy(p->stream);
    if (p->mem) hipFree(p->mem);
    delete p;
}

static dvr_tune default_tune()
{
    dvr_tune t;
    t.wg_per_cu = 4;
    t.xy_tile = 0;
    t.xy_zrun = 32;
    t.z_chunk = 8;
    t.ray_tile = 0;
    return t;
}

static dvr_status check_tune(const dvr_tune &t)
{
    if (t.wg_per_cu < 1 || t.wg_per_cu > 8) return fail(DVR_E_INVALID_ARG, "tune.wg_per_cu must be in [1, 8]");
    if (t.xy_tile < 0 || t.xy_tile > 2) return fail(DVR_E_INVALID_ARG, "tune.xy_tile must be 0, 1 or 2");
    if (t.xy_zrun < 1 || t.xy_zrun > 32) return fail(DVR_E_INVALID_ARG, "tune.xy_zrun must be in [1, 32]");
    if (t.z_chunk < 1 || t.z_chunk > 64) return fail(DVR_E_INVALID_ARG, "tune.z_chunk must be in [1, 64]");
    if (t.ray_tile < 0 || t.ray_tile > 2) return fail(DVR_E_INVALID_ARG, "tune.ray_tile must be 0, 1 or 2");
    return DVR_OK;
}

// Lanes per ray of a view of a batch of `rays` rays.
static int view_lanes(const dvr_batch_desc &d, const KCam &cam, int W, int H, const KGrid &g, double rays)
{
    return fwd_lanes(rays, d.vols[0].feat.layout, d.vols[0].feat.dtype, d.tf.K, view_geo(cam, W, H, g));
}

// Whether a view takes one lane per ray, and so tune.ray_tile has an effect.
static bool has_one_lane(const dvr_batch_desc &d)
{
    double rays = 0.0;
    for (int w = 0; w < d.nview; ++w) rays += (double)d.views[w].cam.width * d.views[w].cam.height;
    for (int w = 0; w < d.nview; ++w) {
        const dvr_batch_view &v = d.views[w];
        if (v.volume < 0 || v.volume >= d.nvol) continue;
        const dvr_grid &vg = d.vols[v.volume].grid;
        KCam cam;
        KGrid g;
        const float h[3] = {vg.hx, vg.hy, vg.hz};
        cam.persp = v.cam.persp;
        for (int k = 0; k < 3; ++k) {
            cam.o[k] = v.cam.o[k];
            cam.d0[k] = v.cam.d0[k];
            cam.du[k] = v.cam.du[k];
            cam.dv[k] = v.cam.dv[k];
        }
        g.n[0] = vg.nx;
        g.n[1] = vg.ny;
        g.n[2] = vg.nz;
        set_grid_steps(g, h, d.rp.step_vox);
        if (view_lanes(d, cam, v.cam.width, v.cam.height, g, rays) == 1) return true;
    }
    return false;
}

static dvr_status create_plan(const dvr_batch_desc *d, dvr_batch **plan_out)
{
    if (!d || !plan_out) return fail(DVR_E_NULL, "desc and plan must be non-NULL");
    *plan_out = nullptr;
    if (d->nvol < 1 || !d->vols) return fail(DVR_E_INVALID_ARG, "need at least one volume");
    if (d->nview < 0 || (d->nview > 0 && !d->views)) return fail(DVR_E_INVALID_ARG, "bad view array");
    const dvr_tune tune = d->tune ? *d->tune : default_tune();
    dvr_status s = check_tune(tune);
    if (s) return s;
    const dvr_feature_params &fp = d->fp;
    if (!(fp.c > 0.f)) return fail(DVR_E_UNSUPPORTED, "batched launches need an explicit Frangi c > 0");
    const int ns = fp.nsigma;
    if ((int64_t)d->nvol * (ns > 0 ? ns : 1) > kMaxVolScale)
        return fail(DVR_E_INVALID_ARG, "volumes x scales must not exceed %d", kMaxVolScale);
    const int layout = d->vols[0].feat.layout, fdt = d->vols[0].feat.dtype;

    size_t lds_floats = 0;  // of the named feature tile (part of the plan's contract: refused above 60 KB)
    std::vector<dvr_features_buf> feats(d->nvol);
    for (int v = 0; v < d->nvol; ++v) {
        const dvr_batch_volume &bv = d->vols[v];
        if ((s = check_grid(&bv.grid))) return fail(s, "volume %d: %s", v, g_err.c_str());
        if ((s = check_fparams(&bv.grid, &fp))) return fail(s, "volume %d: %s", v, g_err.c_str());
        if ((s = check_feat_buf(&bv.feat, true))) return fail(s, "volume %d: %s", v, g_err.c_str());
        if (bv.feat.layout != layout || bv.feat.dtype != fdt)
            return fail(DVR_E_UNSUPPORTED, "all volumes must share the feature dtype and layout");
        if (bv.vol_dtype != fdt) return fail(DVR_E_UNSUPPORTED, "volume %d: vol dtype must equal the feature dtype", v);
        if (!bv.vol || !aligned16(bv.vol)) return fail(bv.vol ? DVR_E_ALIGN : DVR_E_NULL, "volume %d: bad vol pointer", v);
        const double h[3] = {bv.grid.hx, bv.grid.hy, bv.grid.hz};
        for (int sc = 0; sc < ns; ++sc) {
            const int Rx = gauss_radius((double)fp.sigma_mm[sc] / h[0]) + 1, Ry = gauss_radius((double)fp.sigma_mm[sc] / h[1]) + 1;
            lds_floats = std::max(lds_floats, tune.xy_tile == 0   ? xy_lds_floats<64, 8>(Rx, Ry)
                                              : tune.xy_tile == 1 ? xy_lds_floats<32, 16>(Rx, Ry)
                                                                  : xy_lds_floats<128, 4>(Rx, Ry));
        }
        feats[v] = bv.feat;
        feats[v].bricks = nullptr;
    }
    if (lds_floats * 4 > 60 * 1024)
        return fail(DVR_E_UNSUPPORTED, "feature tile with halo needs %zu bytes of LDS (limit 60 KB)", lds_floats * 4);
    // views
    std::vector<BView> views(d->nview);
    double rays = 0.0;
    RayArgs A;
    memset(&A, 0, sizeof A);
    for (int w = 0; w <= d->nview; ++w) {
        // the TF and the render parameters are checked (and taken) on a dummy view, also without views
        dvr_batch_view bw;
        memset(&bw, 0, sizeof bw);
        bw.cam.width = bw.cam.height = 1;
        bw.cam.d0[2] = 1.f;
        if (w < d->nview) bw = d->views[w];
        if (bw.volume < 0 || bw.volume >= d->nvol) return fail(DVR_E_INVALID_ARG, "view %d: bad volume index", w);
        const dvr_batch_volume &bv = d->vols[bw.volume];
        dvr::RenderArgs ra;
        dvr::KCam kc;
        if ((s = build_render_args(bv.vol, bv.vol_dtype, &bv.grid, &bv.feat, &d->tf, &d->rp, &bw.cam, 1, ra, &kc)))
            return w < d->nview ? fail(s, "view %d: %s", w, g_err.c_str()) : s;
        if (w == d->nview) {
            A.tf = ra.tf;
            A.rp = ra.rp;
            break;
        }
        if (!bw.rgba || !aligned16(bw.rgba)) return fail(bw.rgba ? DVR_E_ALIGN : DVR_E_NULL, "view %d: bad rgba", w);
        BView &V = views[w];
        V.cam = kc;
        V.feat = ra.feat;
        V.grid = ra.grid;
        V.W = bw.cam.width;
        V.H = bw.cam.height;
        V.need = 1u;
        V.rgba = bw.rgba;
        V.T_last = bw.T_last;
        V.k_last = bw.T_last ? bw.k_last : nullptr;
        rays += (double)V.W * V.H;
    }
    // Test hook (DVR_BATCH_TEST_TIMEOUT=1): the rays of volume 0 wait for a stage that never comes, with a
    // short bound, so the launch exercises the timeout path and still exits normally.
    A.max_spin = kMaxSpin;
    if (getenv("DVR_BATCH_TEST_TIMEOUT") && atoi(getenv("DVR_BATCH_TEST_TIMEOUT")) == 1) {
        for (int w = 0; w < d->nview; ++w)
            if (d->views[w].volume == 0) views[w].need = 2u;
        A.max_spin = 2000;
    }
    // the ray tables, one for each number of lanes per ray: workgroup b is XCD b % 8's, and the blocks of
    // 2 x 2 tiles go to the XCDs in turn
    const int lanes_of[3] = {1, 4, 16};
    std::vector<BBlock> blocks[3];
    for (int q = 0; q < 3; ++q) {
        std::vector<BBlock> xcd[8];
        int64_t turn = 0;
        for (int w = 0; w < d->nview; ++w) {
            const BView &V = views[w];
            if (view_lanes(*d, V.cam, V.W, V.H, V.grid, rays) != lanes_of[q]) continue;
            const int S = (int)tile_side(lanes_of[q]), nx = (V.W + S - 1) / S, ny = (V.H + S - 1) / S;
            for (int by = 0; by < ny; by += 2)
                for (int bx = 0; bx < nx; bx += 2, ++turn)
                    xcd[(turn + 5 * (turn >> 3) + (turn >> 6) + (turn >> 9)) & 7].push_back({w, bx, by, 0});
        }
        size_t most = 0;
        for (const auto &x : xcd) most = std::max(most, x.size());
        if (most * 8 > 0x7fffffffu) return fail(DVR_E_INVALID_ARG, "too many work items");
        blocks[q].assign(most * 8, BBlock{-1, 0, 0, 0});
        for (size_t x = 0; x < 8; ++x)
            for (size_t i = 0; i < xcd[x].size(); ++i) blocks[q][i * 8 + x] = xcd[x][i];
    }
    // The features as units of work: a large volume, or small ones whose passes share launches (features_group.hip)
    std::vector<Unit> units;
    std::vector<Unit> small;
    for (int v = 0; v < d->nvol; ++v) {
        const int64_t n = nvox(&d->vols[v].grid);
        if (!groupable(d->vols[v].grid, fp)) {
            units.push_back({n, {v}});
            continue;
        }
        if (small.empty() || small.back().vox + n > kGroupSum) small.push_back({0, {}});
        small.back().vox += n;
        small.back().vols.push_back(v);
    }
    for (Unit &u : small) u.shared = u.vols.size() > 1 || too_tall(d->vols[u.vols[0]].grid);
    units.insert(units.end(), small.begin(), small.end());
    // on branches (one alone leaves CUs idle): largest first to the least loaded, a workspace per branch
    const int nlane = std::min(kLanes, (int)units.size());
    std::sort(units.begin(), units.end(), [](const Unit &a, const Unit &b) {
        return a.vox > b.vox || (a.vox == b.vox && a.vols[0] < b.vols[0]);
    });
    int64_t load[kLanes] = {}, ws_vox[kLanes] = {};
    for (Unit &u : units) {
        for (int k = 1; k < nlane; ++k) u.lane = load[k] < load[u.lane] ? k : u.lane;
        load[u.lane] += u.vox;
        ws_vox[u.lane] = std::max(ws_vox[u.lane], u.vox);
    }

    dvr_batch *P = new (std::nothrow) dvr_batch();
    if (!P) return fail(DVR_E_NOMEM, "host allocation");
    std::unique_ptr<dvr_batch, void (*)(dvr_batch *)> own(P, plan_free);
    P->tune = tune;
    // the groups' launches: their table holds a row for each volume, scale and pass (workspaces from 0 for now)
    std::vector<FeatItem> items;
    std::vector<GroupRun> runs;
    for (size_t u = 0; u < units.size(); ++u)
        if (units[u].shared) group_runs(*d, feats, (int)u, units[u], items, runs);
    std::vector<float *> gmax(d->nvol);
    for (int v = 0; v < d->nvol; ++v) gmax[v] = d->vols[v].feat.gmax;
    // one allocation: the tables, which one copy fills, then the stage word and the workspaces
    size_t bytes = 0;
    auto place = [&](size_t n) {
        const size_t at = bytes;
        bytes += (n + 255) & ~(size_t)255;
        return at;
    };
    const size_t at_views = place(sizeof(BView) * views.size()), at_gmax = place(sizeof(float *) * gmax.size()),
                 at_items = place(sizeof(FeatItem) * items.size());
    size_t at_blocks[3], at_ws[kLanes];
    for (int q = 0; q < 3; ++q) at_blocks[q] = place(sizeof(BBlock) * blocks[q].size());
    std::vector<char> tables(bytes);
    const size_t at_ctr = place(256);
    for (int l = 0; l < nlane; ++l) at_ws[l] = place(12u * (size_t)ws_vox[l]);
    if (hipMalloc((void **)&P->mem, bytes) != hipSuccess) {
        P->mem = nullptr;
        return fail(DVR_E_DEVICE, "device allocation of %zu bytes of workspace failed", bytes);
    }
    for (const GroupRun &g : runs)
        for (int i = 0; i < g.count; ++i) {
            XYArgs &a = items[g.first + i].a;
            a.ws = (const float *)(P->mem + at_ws[units[g.unit].lane] + (size_t)(uintptr_t)a.ws);
        }
    auto fill = [&](size_t at, const void *src, size_t n) {
        if (n) memcpy(tables.data() + at, src, n);
    };
    fill(at_views, views.data(), sizeof(BView) * views.size());
    fill(at_gmax, gmax.data(), sizeof(float *) * gmax.size());
    fill(at_items, items.data(), sizeof(FeatItem) * items.size());
    for (int q = 0; q < 3; ++q) fill(at_blocks[q], blocks[q].data(), sizeof(BBlock) * blocks[q].size());
    float **d_gmax = (float **)(P->mem + at_gmax);
    const FeatItem *d_items = (const FeatItem *)(P->mem + at_items);
    A.views = (uint64_t)(uintptr_t)(P->mem + at_views);
    A.ray_tile = tune.ray_tile;
    A.stage = (unsigned *)(P->mem + at_ctr);
    A.err = A.stage + 1;
    P->d_err = A.err;
    hipError_t e = hipMemcpy(P->mem, tables.data(), tables.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&P->stream, hipStreamNonBlocking);
    if (e != hipSuccess) {
        return dev_fail(e, "batch plan setup");
    }
    e = hipStreamBeginCapture(P->stream, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        auto record = [&]() -> hipError_t {
            hipError_t r;
            hipLaunchKernelGGL(k_batch_init, dim3(1), dim3(256), 0, P->stream, A.stage, A.err, d_gmax, d->nvol);
            if ((r = hipGetLastError()) != hipSuccess) return r;
            // the branches are recorded one after the other on the one capturing stream, each from the
            // init node on; then the stream goes on from their last nodes
            std::vector<hipGraphNode_t> head, tails;
            if ((r = capture_tail(P->stream, head)) != hipSuccess) return r;
            for (int l = 0; l < nlane; ++l) {
                if ((r = hipStreamUpdateCaptureDependencies(P->stream, head.data(), head.size(),
                                                            hipStreamSetCaptureDependencies)) != hipSuccess)
                    return r;
                for (size_t u = 0; u < units.size(); ++u) {
                    if (units[u].lane != l) continue;
                    if (!units[u].shared) {
                        const int v = units[u].vols[0];
                        const dvr_batch_volume &bv = d->vols[v];
                        if ((r = enqueue_features(bv.vol, bv.vol_dtype, &bv.grid, &fp, &feats[v], nullptr, (float *)(P->mem + at_ws[l]),
                                                  P->stream)) != hipSuccess)
                            return r;
                    }
                    for (const GroupRun &g : runs)
                        if (g.unit == (int)u && (r = launch_run(g, d_items, fdt, layout, P->stream)) != hipSuccess) return r;
                }
                if ((r = capture_tail(P->stream, tails)) != hipSuccess) return r;
            }
            if ((r = hipStreamUpdateCaptureDependencies(P->stream, tails.data(), tails.size(),
                                                        hipStreamSetCaptureDependencies)) != hipSuccess)
                return r;
            hipLaunchKernelGGL(k_batch_mark, dim3(1), dim3(64), 0, P->stream, A.stage);
            if ((r = hipGetLastError()) != hipSuccess) return r;
            for (int q = 0; q < 3; ++q) {
                // a table of more tiles than one grid holds takes several launches, each of whole rounds of
                // the 8 XCDs
                const size_t per = kMaxGroups / 32 * 8;
                for (size_t b = 0; b < blocks[q].size(); b += per) {
                    A.blocks = (uint64_t)(uintptr_t)(P->mem + at_blocks[q] + sizeof(BBlock) * b);
                    const size_t n = std::min(per, blocks[q].size() - b);
                    if ((r = launch_rays(A, layout, fdt, lanes_of[q], (unsigned)(4 * n), P->stream)) != hipSuccess) return r;
                }
            }
            return hipSuccess;
        };
        const hipError_t e1 = record();
        const hipError_t e2 = hipStreamEndCapture(P->stream, &P->graph);
        e = e1 != hipSuccess ? e1 : e2;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&P->exec, P->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        return dev_fail(e, "batch graph capture");
    }
    *plan_out = own.release();
    return DVR_OK;
}

extern "C" dvr_status dvr_batch_create(const dvr_batch_desc *d, dvr_batch **plan_out)
{
    try {
        return create_plan(d, plan_out);
    } catch (const std::exception &) {  // the tables' std::bad_alloc
        return fail(DVR_E_NOMEM, "host allocation");
    }
}

extern "C" dvr_status dvr_batch_launch(dvr_batch *plan, hipStream_t stream)
{
    if (!plan || !plan->exec) return fail(DVR_E_NULL, "plan is NULL");
    const hipError_t e = hipGraphLaunch(plan->exec, stream);
    return e == hipSuccess ? DVR_OK : dev_fail(e, "batch graph launch");
}

extern "C" dvr_status dvr_batch_check(dvr_batch *plan, hipStream_t stream)
{
    if (!plan) return fail(DVR_E_NULL, "plan is NULL");
    hipError_t e = hipStreamSynchronize(stream);
    unsigned err = 0;
    if (e == hipSuccess) e = hipMemcpy(&err, plan->d_err, sizeof err, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return dev_fail(e, "batch check");
    if (err) return fail(DVR_E_TIMEOUT, "a dependency wait of the batched launch expired");
    return DVR_OK;
}

extern "C" dvr_status dvr_batch_destroy(dvr_batch *plan)
{
    if (!plan) return DVR_OK;
    hipStreamSynchronize(plan->stream);
    plan_free(plan);
    return DVR_OK;
}

// ------------------------------------------------------------------------------------------------
// autotuner: times the ray tiles on the batch itself; JSON cache keyed by shape class

// Batches whose views all share a ray among lanes, where no field has an effect, have keys of their own: their
// entry says nothing about a batch of the same class with finer views.
static std::string tune_key(const dvr_batch_desc *d, bool one_lane)
{
    double vox = 0, pix = 0;
    for (int v = 0; v < d->nvol; ++v) vox += (double)nvox(&d->vols[v].grid);
    for (int w = 0; w < d->nview; ++w) pix += (double)d->views[w].cam.width * d->views[w].cam.height;
    int dev = 0;
    hipGetDevice(&dev);
    hipDeviceProp_t prop;
    std::string arch = "gpu";
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess) arch = prop.gcnArchName;
    std::ostringstream k;
    k << arch.substr(0, arch.find(':')) << "|dt" << d->vols[0].feat.dtype << "|lay" << d->vols[0].feat.layout << "|ns"
      << d->fp.nsigma << "|K" << (d->tf.K <= 16 ? 16 : 64) << "|vox2^" << (int)floor(log2(std::max(vox, 1.0)))
      << "|pix2^" << (int)floor(log2(std::max(pix, 1.0))) << "|nvol2^" << (int)floor(log2((double)d->nvol))
      << (one_lane ? "" : "|shared");
    return k.str();
}

static std::map<std::string, dvr_tune> read_cache(const char *path)
{
    std::map<std::string, dvr_tune> m;
    std::ifstream f(path);
    std::string line;
    while (std::getline(f, line)) {
        // "key": [wg_per_cu, xy_tile, xy_zrun, z_chunk, ray_tile],
        const size_t q0 = line.find('"'), q1 = line.find('"', q0 + 1), b0 = line.find('['), b1 = line.find(']');
        if (q0 == std::string::npos || q1 == std::string::npos || b0 == std::string::npos || b1 == std::string::npos)
            continue;
        dvr_tune t;
        if (sscanf(line.c_str() + b0 + 1, "%d , %d , %d , %d , %d", &t.wg_per_cu, &t.xy_tile, &t.xy_zrun, &t.z_chunk,
                   &t.ray_tile) == 5 &&
            check_tune(t) == DVR_OK)
            m[line.substr(q0 + 1, q1 - q0 - 1)] = t;
    }
    return m;
}

static void write_cache(const char *path, const std::map<std::string, dvr_tune> &m)
{
    std::ofstream f(path);
    f << "{\n";
    size_t i = 0;
    for (const auto &kv : m) {
        const dvr_tune &t = kv.second;
        f << "  \"" << kv.first << "\": [" << t.wg_per_cu << ", " << t.xy_tile << ", " << t.xy_zrun << ", " << t.z_chunk
          << ", " << t.ray_tile << "]" << (++i < m.size() ? "," : "") << "\n";
    }
    f << "}\n";
}

// Times the three ray tiles on the batch; best_t: the defaults, then the fastest.  (The default feature tile's
// halo fits at every radius, so no candidate is refused where a plan is not.)
static dvr_status time_ray_tiles(const dvr_batch_desc &desc, dvr_tune &best_t)
{
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) hipEventDestroy(e0);
        return fail(DVR_E_DEVICE, "event creation");
    }
    dvr_status last = DVR_OK;
    float best_ms = INFINITY;
    for (int r = 0; r < 3; ++r) {
        dvr_tune t = default_tune();
        t.ray_tile = r;
        // one candidate: build the plan, one warm replay, then two timed replays
        dvr_batch_desc d = desc;
        d.tune = &t;
        dvr_batch *p = nullptr;
        last = dvr_batch_create(&d, &p);
        if (last != DVR_OK) break;
        float ms = INFINITY;
        if (dvr_batch_launch(p, p->stream) == DVR_OK && dvr_batch_check(p, p->stream) == DVR_OK) {
            hipEventRecord(e0, p->stream);
            dvr_batch_launch(p, p->stream);
            dvr_batch_launch(p, p->stream);
            hipEventRecord(e1, p->stream);
            if (dvr_batch_check(p, p->stream) != DVR_OK || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) ms = INFINITY;
        }
        dvr_batch_destroy(p);
        if (ms < best_ms) {
            best_ms = ms;
            best_t = t;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (last != DVR_OK) return last;
    return isfinite(best_ms) ? DVR_OK : fail(DVR_E_DEVICE, "no candidate tune ran");
}

static dvr_status autotune(const dvr_batch_desc *desc, const char *cache_path, dvr_tune *best)
{
    if (!desc || !best) return fail(DVR_E_NULL, "desc and best must be non-NULL");
    if (desc->nvol < 1 || !desc->vols) return fail(DVR_E_INVALID_ARG, "need at least one volume");
    if (desc->nview < 0 || (desc->nview > 0 && !desc->views)) return fail(DVR_E_INVALID_ARG, "bad view array");
    const bool one_lane = has_one_lane(*desc);
    const std::string key = tune_key(desc, one_lane);
    std::map<std::string, dvr_tune> cache;
    if (cache_path) {
        cache = read_cache(cache_path);
        auto it = cache.find(key);
        if (it != cache.end()) {
            *best = it->second;
            return DVR_OK;
        }
    }
    dvr_tune best_t = default_tune();
    if (!one_lane) {
        // nothing to choose: a plan is built for its checks alone
        dvr_batch_desc d = *desc;
        d.tune = &best_t;
        dvr_batch *p = nullptr;
        const dvr_status s = dvr_batch_create(&d, &p);
        if (s != DVR_OK) return s;
        dvr_batch_destroy(p);
    } else {
        const dvr_status s = time_ray_tiles(*desc, best_t);
        if (s != DVR_OK) return s;
    }
    *best = best_t;
    if (cache_path) {
        cache[key] = best_t;
        write_cache(cache_path, cache);
    }
    return DVR_OK;
}

extern "C" dvr_status dvr_batch_autotune(const dvr_batch_desc *desc, const char *cache_path, dvr_tune *best)
{
    try {
        return autotune(desc, cache_path, best);
    } catch (const std::exception &) {
        return fail(DVR_E_NOMEM, "host allocation");
    }
}
