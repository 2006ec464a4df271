// Front-to-back raymarcher (Sec. 2.4 Eq. 4-6) and its adjoint, for gfx950.
//
// Mapping: one lane per ray, or 4 or 16 where the rays are few or coarse (lanes.hpp); with one a wave
// covers an 8 x 8 pixel tile and a 256-lane workgroup a 16 x 16 tile, so the lanes of a wave gather
// neighbouring voxels.  A lane leaves the sample loop when its ray ends or terminates early; the wave
// leaves when every lane has (the exec mask of the loop empties), which is the wave-ballot early
// termination.
//
// Ray geometry.  The camera ray, the slab clip against [0,(n-1)h] and the segment count are
// computed once per ray in double-float FP32 (pairs of FP32 numbers, ~48 bits, from error-free
// transforms), following the FP64 definition's steps, so N and the segment lengths agree with it
// (plain FP32 here moves the head's perspective images by ~6e-4).  Sample positions in voxel units
// are then carried in 32.32 fixed point: q_k = q_0 + k dq for the full segments and the midpoint
// of the shorter last segment separately.  Integer steps are exact and reversible, so the adjoint
// walks the same positions back to front, and the clamp of the first and last positions (plus a
// one-time check of the last full step) keeps every cell index inside [0, n-2] without per-sample
// clamping.  FP32 positions would be off by up to 1e-4 voxel at a perspective camera two box
// diagonals away, which moves the image by more than the 1e-5 parity budget.
//
// Per sample: trilinear I (8 gathers); the TF segment (knots in scalar registers, values and
// slopes in LDS); when the extinction is zero the sample is exactly transparent and the feature
// gathers are skipped; otherwise g, k, V (planar: 5 x 8 gathers; interleaved record: the same
// loads merged), Eq. 4 factors, alpha = -expm1(-sigma delta_k), C += T alpha c, T *= 1 - alpha.
#include <math.h>

#include "common.hpp"
#include "lanes.hpp"
#include "render_args.hpp"
#include "render_dev.hpp"

namespace dvr {

// ------------------------------------------------------------------------------------------------
// The camera index is uniform over the workgroup; copying the record field by field keeps the
// by-value kernel argument block in the constant segment (taking its address would make the
// compiler copy the whole block to per-lane scratch).
__device__ __forceinline__ KCam load_cam(const KLaunch &L, uint32_t cam)
{
    cam = __builtin_amdgcn_readfirstlane(cam);
    KCam c;
    c.persp = L.cams[cam].persp;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        c.o[a] = L.cams[cam].o[a];
        c.d0[a] = L.cams[cam].d0[a];
        c.du[a] = L.cams[cam].du[a];
        c.dv[a] = L.cams[cam].dv[a];
    }
    return c;
}

// Camera and pixel of this lane's ray in the workgroup's tile: 16 x 16 pixels of which a wave takes 8 x 8,
// or, with G = 4 or 16 lanes per ray, 8 x 8 and 4 x 4 or 4 x 4 and 2 x 2.
//
// Which tile a workgroup takes decides what its XCD's L2 holds and how even the XCDs' loads are:
// consecutive workgroups go to different XCDs, each with an L2 of its own.  Views in multiples of eight:
// each XCD takes a contiguous eighth of the launch, whole views, row by row.  Otherwise (L.spread) that
// gives rows of background to some XCDs and the whole object to others, so the tiles are grouped into
// blocks of 2 x 2, which the XCDs take in turn, rotated from one round of eight to the next so that none
// keeps a column of the image or the centre of every view: one 1024^2 view of a head 0.81 -> 0.55 ms, two
// 2048^2 views of a 512 x 512 x 400 volume 14.2 -> 7.9.  Eight views are within 5 % either way, so whole
// views stay: the head 2.68 ms as whole views, 2.78 dealt out; eight 2048^2 views of the 512 x 512 x 400 volume
// 30.2, 28.9; training steps on it at 1024^2 31.1, 31.9, on a 128^3 volume 5.92, 5.99.
//
// MORTON: a wave's rays take their pixels in Morton order (bits x0 y0 x1 y1 x2 y2), so each quad of lanes
// (G = 1) is a 2 x 2 pixel block and each row of 16 a 4 x 4 one; otherwise row-major.
template <bool MORTON = false, int G = 1>
__device__ __forceinline__ void pixel_of(const KLaunch &L, uint32_t &cam, int &pi, int &pj, bool &valid)
{
    constexpr uint32_t S = tile_side(G);
    // one form for both (blocks of one tile in contiguous eighths): a branch here, though uniform and not
    // taken, made the whole kernel 2.5 % slower on eight head views
    const uint32_t sp = L.spread, lg = (G == 1 ? 4u : (G == 4 ? 3u : 2u)) + sp;
    const uint32_t bx = ((uint32_t)L.W + (1u << lg) - 1u) >> lg, by = ((uint32_t)L.H + (1u << lg) - 1u) >> lg;
    const uint32_t i = blockIdx.x >> 3, round = i >> (2u * sp), w = i & ((1u << (2u * sp)) - 1u);
    const uint32_t turn = round * 8u + ((blockIdx.x + 5u * round + (round >> 3) + (round >> 6)) & 7u);
    const uint32_t blk = sp ? turn : (blockIdx.x & 7u) * (gridDim.x >> 3) + round;
    cam = blk / (bx * by);
    const uint32_t bb = blk - cam * (bx * by);
    const uint32_t b_y = bb / bx, b_x = bb - b_y * bx;
    const uint32_t tx = (b_x << sp) + (w & 1u), ty = (b_y << sp) + (w >> 1);
    const uint32_t lane = (threadIdx.x & 63u) / G, wv = threadIdx.x >> 6;
    uint32_t lx, ly;
    if (MORTON) {
        lx = (lane & 1u) | ((lane >> 1) & 2u) | ((lane >> 2) & 4u);
        ly = ((lane >> 1) & 1u) | ((lane >> 2) & 2u) | ((lane >> 3) & 4u);
    } else {
        lx = lane % (S / 2);
        ly = lane / (S / 2);
    }
    pi = (int)(tx * S + (wv & 1u) * (S / 2) + lx);
    pj = (int)(ty * S + (wv >> 1) * (S / 2) + ly);
    valid = cam < (uint32_t)L.ncam && pi < L.W && pj < L.H;
}

// The FP16 quad layout keeps a corner's six values packed in three registers (104 VGPRs, four waves
// per SIMD); held to five waves (96 VGPRs, a few spilled values) it runs 7 % faster on the head
// (0.296 against 0.318 ms per view).  The FP32 layouts and the other FP16 ones spill far more at
// five waves and are slower, so they keep the default.
// G: lanes per ray.
template <int LAYOUT, int DT, int KMAX, int G>
__global__ __launch_bounds__(256, (LAYOUT == DVR_QUAD && DT == DVR_F16 && G == 1) ? 5 : 1) void k_render(
    KFeat feat, KGrid g, KTF tf, KRender rp, KLaunch L)
{
    __shared__ TFShared<KMAX> sh;
    float kx[KMAX];
    tf_load<KMAX>(sh, kx, tf);
    __syncthreads();
    uint32_t cam;
    int pi, pj;
    bool valid;
    pixel_of<false, G>(L, cam, pi, pj, valid);
    const float gm = *feat.gmax;
    const float invg = gm > 0.f ? 1.f / gm : 0.f;
    RayGeo r;
    r.N = 0;
    if (valid) r = ray_setup(load_cam(L, cam), pi, pj, g);
    RayOut o;
    if constexpr (G == 1) o = march_fwd<LAYOUT, DT, KMAX>(feat, g, sh, kx, rp, invg, r);
    else o = march_fwd_group<LAYOUT, DT, KMAX, G>(feat, g, sh, kx, rp, invg, r);
    const bool first = G == 1 || (threadIdx.x & (G - 1)) == 0;  // one lane of the group writes
    if (valid && first) {
        const size_t pix = ((size_t)(L.cam_base + cam) * L.H + pj) * L.W + pi;
        reinterpret_cast<float4 *>(L.out)[pix] = make_float4(o.C0, o.C1, o.C2, o.A);
        if (L.T_last) L.T_last[pix] = o.Tprev;
        if (L.k_last) L.k_last[pix] = o.last;
    }
    if (L.counters) count_samples<4>(L.counters, first ? o.last : -1, o.shaded);
}

// Gather ceiling of k_render (dvr_render_gather): the same rays, samples and loads, without the
// optics; sink[pixel] keeps the loads live, counters count the samples walked and those whose
// feature corners were fetched (equal to the forward pass's counts by construction).
template <int LAYOUT, int DT, int KMAX>
__global__ __launch_bounds__(256) void k_render_gather(KFeat feat, KGrid g, KTF tf, KRender rp, KLaunch L)
{
    __shared__ TFShared<KMAX> sh;
    float kx[KMAX];
    tf_load<KMAX>(sh, kx, tf);
    __syncthreads();
    uint32_t cam;
    int pi, pj;
    bool valid;
    pixel_of(L, cam, pi, pj, valid);
    const size_t pix = valid ? ((size_t)(L.cam_base + cam) * L.H + pj) * L.W + pi : 0;
    const int kl = valid ? L.k_last[pix] : -1;
    RayGeo r;
    r.N = 0;
    if (kl >= 0) r = ray_setup(load_cam(L, cam), pi, pj, g);
    const RayOut o = march_fwd<LAYOUT, DT, KMAX, true>(feat, g, sh, kx, rp, 0.f, r, kl);
    if (valid) L.out[pix] = o.C0;
    if (L.counters) count_samples<4>(L.counters, o.last, o.shaded);
}

// value of another lane of the wave
__device__ __forceinline__ int64_t shfl64(int64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, lane, 64), hi = (uint32_t)__shfl((int)(v >> 32), lane, 64);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Adjoint of a 16 x 16 pixel tile per workgroup, 8 x 8 pixels per wave.  G = 1: one lane per ray
// (march_bwd).  G = 4, 16: G lanes per ray (march_bwd_group), the wave's 64 rays in G blocks of 64 / G
// (4 x 4 or 2 x 2 pixels) taken one after another; every lane sets one ray up and the blocks read
// theirs from it, so the set-up is not repeated within a group.  The blocks of a tile may be dealt to
// several workgroups (gridDim.y).
// Per call, render adjoint with feature gradients / plain, G = 1 against 4 (pitch in voxels a pixel):
// head 1024^2 x 2 (0.35) 8.3 -> 9.7 / 3.8 -> 4.4 ms, 128^3 512^2 x 4 (0.43) 11.4 -> 7.4 / 2.3 -> 2.5, head
// 512^2 x 2 (0.70) 5.7 -> 2.7 / 1.52 -> 1.37, 128^3 256^2 x 4 (0.86) 18.1 -> 2.7 / 2.5 -> 0.79; against 16:
// 172 x 373 x 89, 231 x 286 x 6 (1.8) 28.0 -> 7.5 / 5.7 -> 1.75, 128^3 128^2 x 2 (1.7) 5.9 -> 1.1 / 2.0 -> 0.30.
template <int LAYOUT, int DT, int KMAX, bool FG, int G>
__global__ __launch_bounds__(256) void k_render_bwd(KFeat feat, KGrid g, KTF tf, KRender rp, KLaunch L)
{
    __shared__ TFShared<KMAX> sh;
    constexpr int kCopies = tf_copies(KMAX);
    __shared__ double tfa[KMAX * 4 * kCopies];
    using Win = DWinG<FG, G>;
    __shared__ double win[4][Win::kEntries];  // one accumulation window per wave
    // the ray first, before anything else is live: set up after the TF load (with the knots held in
    // registers across it) the kernel took 182 VGPRs instead of 166, one wave per SIMD fewer
    uint32_t cam;
    int pi, pj;
    bool valid;
    pixel_of<true>(L, cam, pi, pj, valid);
    const int pix = valid ? (int)(((size_t)(L.cam_base + cam) * L.H + pj) * L.W + pi) : -1;
    const int kl = valid ? L.k_last[pix] : -1;
    const int nb = G / (int)gridDim.y;  // blocks of this workgroup
    if constexpr (G > 1) {
        // a workgroup without a live ray ends here, before it clears its window (98 KB with feature
        // gradients and 16 lanes): a 231 x 286 x 6 volume in the middle of four 512^2 views of 5 voxels a
        // pixel 0.50 -> 0.20 ms (plain 0.24 -> 0.11; with one lane a ray 0.32 and 0.17)
        // (__syncthreads_or here: 170 VGPRs instead of 166, one wave per SIMD fewer, 7 % slower)
        __shared__ uint32_t alive[4];
        const uint64_t mine = __ballot(kl >= 0 && (int)(threadIdx.x & 63u) / (64 / G) / nb == (int)blockIdx.y);
        if ((threadIdx.x & 63u) == 0) alive[threadIdx.x >> 6] = mine != 0;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(alive[0] | alive[1] | alive[2] | alive[3]) == 0) return;
    }
    RayGeo r;
    r.N = 0;
    if (kl >= 0) r = ray_setup(load_cam(L, cam), pi, pj, g);
    float kx[KMAX];
    tf_load<KMAX>(sh, kx, tf);
    for (int p = threadIdx.x; p < KMAX * 4 * kCopies; p += 256) tfa[p] = 0.0;
    double *wwin = win[threadIdx.x >> 6];
    if (FG || L.dvol)
        for (int p = threadIdx.x & 63; p < Win::kEntries; p += 64) wwin[p] = 0.0;
    __syncthreads();
    const int K = tf.K;
    const float gm = *feat.gmax;
    const float invg = gm > 0.f ? 1.f / gm : 0.f;
    double *tfl = tfa + (threadIdx.x % kCopies);
    float gmb = 0.f;
    if constexpr (G == 1) {
        float4 gr = make_float4(0.f, 0.f, 0.f, 0.f);
        float Tl = 0.f;
        if (kl >= 0) {
            gr = reinterpret_cast<const float4 *>(L.dout)[pix];
            Tl = L.T_last[pix];
        }
        // every lane of the wave takes part (the dL/dI window is managed wave-wide)
        march_bwd<LAYOUT, DT, KMAX, FG>(feat, g, sh, kx, rp, invg, r, kl, Tl, gr, K, tfl, L.dvol, wwin, L.dfeat, gmb);
    } else {
        for (int blk = (int)blockIdx.y * nb; blk < ((int)blockIdx.y + 1) * nb; ++blk) {
            const int src = blk * (64 / G) + (int)(threadIdx.x & 63u) / G;
            const int k1 = __shfl(kl, src, 64);
            if (!__any(k1 >= 0)) continue;
            GroupRay q;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                q.q0[a] = shfl64(r.q0[a], src);
                q.dq[a] = shfl64(r.dq[a], src);
                q.ql[a] = shfl64(r.ql[a], src);
            }
            q.N = __shfl(r.N, src, 64);
            q.delta = g.delta_hi;
            q.dlast = __shfl(r.dlast, src, 64);
            const int px = __shfl(pix, src, 64);
            float4 gr = make_float4(0.f, 0.f, 0.f, 0.f);
            float Tl = 0.f;
            if (k1 >= 0) {
                gr = reinterpret_cast<const float4 *>(L.dout)[px];
                Tl = L.T_last[px];
            }
            march_bwd_group<LAYOUT, DT, KMAX, FG, G, Win>(feat, g, sh, kx, rp, invg, q, k1, Tl, gr, K, tfl, L.dvol, wwin,
                                                          L.dfeat, gmb);
        }
    }
    __shared__ float gw[4];
    if constexpr (FG) {
        for (int o = 32; o > 0; o >>= 1) gmb += __shfl_xor(gmb, o, 64);
        if ((threadIdx.x & 63) == 0) gw[threadIdx.x >> 6] = gmb;
    }
    __syncthreads();
    if constexpr (FG) {  // one add a workgroup: each rounds the one FP32 word
        const double acc = ((double)gw[0] + gw[1]) + ((double)gw[2] + gw[3]);
        if (threadIdx.x == 0 && acc != 0.0) atomicAdd(L.dgmax, (float)acc);
    }
    for (int p = threadIdx.x; p < K * 4; p += 256) {
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < kCopies; ++j) acc += tfa[p * kCopies + j];
        if (acc != 0.0) atomicAdd(L.dtf + p, (float)acc);
    }
}

// ------------------------------------------------------------------------------------------------
enum { kFwd = 0, kBwd = 1, kGather = 2 };

template <int LAYOUT, int DT, int KMAX>
static hipError_t launch_fwd_t(const KFeat &f, const KGrid &g, const KTF &tf, const KRender &rp, const KLaunch &L,
                               hipStream_t st, int mode, const RaySplit &split)
{
    const int lanes = split.lanes;
    const uint32_t blocks = (uint32_t)tile_groups(L.W, L.H, L.ncam, mode == kFwd ? lanes : 1, L.spread);
#define DVR_BWD(FG, G) \
    hipLaunchKernelGGL((k_render_bwd<LAYOUT, DT, KMAX, FG, G>), dim3(blocks, split.parts), dim3(256), 0, st, f, g, tf, rp, L)
    if (mode == kGather) {
        hipLaunchKernelGGL((k_render_gather<LAYOUT, DT, KMAX>), dim3(blocks), dim3(256), 0, st, f, g, tf, rp, L);
    } else if (mode == kFwd) {
        if (lanes == 16)
            hipLaunchKernelGGL((k_render<LAYOUT, DT, KMAX, 16>), dim3(blocks), dim3(256), 0, st, f, g, tf, rp, L);
        else if (lanes == 4)
            hipLaunchKernelGGL((k_render<LAYOUT, DT, KMAX, 4>), dim3(blocks), dim3(256), 0, st, f, g, tf, rp, L);
        else
            hipLaunchKernelGGL((k_render<LAYOUT, DT, KMAX, 1>), dim3(blocks), dim3(256), 0, st, f, g, tf, rp, L);
    } else if (L.dfeat) {
        if (lanes == 16) DVR_BWD(true, 16);
        else if (lanes == 4) DVR_BWD(true, 4);
        else DVR_BWD(true, 1);
    } else {
        if (lanes == 16) DVR_BWD(false, 16);
        else if (lanes == 4) DVR_BWD(false, 4);
        else DVR_BWD(false, 1);
    }
#undef DVR_BWD
    return hipGetLastError();
}

template <int LAYOUT, int DT>
static hipError_t launch_k(const KFeat &f, const KGrid &g, const KTF &tf, const KRender &rp, const KLaunch &L,
                           hipStream_t st, int mode, const RaySplit &split)
{
    if (tf.K <= 8) return launch_fwd_t<LAYOUT, DT, 8>(f, g, tf, rp, L, st, mode, split);
    if (tf.K <= 16) return launch_fwd_t<LAYOUT, DT, 16>(f, g, tf, rp, L, st, mode, split);
    return launch_fwd_t<LAYOUT, DT, 64>(f, g, tf, rp, L, st, mode, split);
}

// Lanes per ray of the adjoint.  Above about 0.4 voxels a pixel the 8 x 8 rays of a wave stop fitting its
// window (feature gradients; 0.65 without them, whose window is larger and whose G = 1 form keeps its
// corner cache), above about 1.5 the 4 x 4 ones do.  Few rays take more lanes whatever the pitch: 64^3
// at 256^2 has 1024 waves for 1024 SIMDs with one lane a ray.
static int bwd_lanes(const KLaunch &L, double pitch)
{
    const double rays = (double)L.W * L.H * L.ncam;
    if (pitch > 1.5 || rays <= 32768.0) return 16;
    if (pitch > (L.dfeat ? 0.39 : 0.65) || rays <= 131072.0) return 4;
    return 1;
}

// Workgroups that share a tile of the adjoint, which evens the load out.  Every one with a live ray adds to the
// same few FP32 words of the TF gradient (and to dL/d|g|_max), and each add rounds them, so there are at most
// about 1024 such workgroups, or twice as many as tiles: relative error of the TF gradient (mean and largest of
// nine runs) of a 114 x 60 x 453 volume in six 184 x 194 views, 217 such tiles, one lane per ray 1.9e-7, 2.6e-7; 1 /
// 4 / 8 / 16 workgroups a tile 0.6e-7, 2.1e-7, 5.5e-7, 6.1e-7 in 4.01 / 3.65 / 3.60 / 3.56 ms; of two 512^2
// views of a head, 706 tiles, 7.2e-7, 1.4e-6; 1 / 2 / 4 a tile 4.5e-7, 3.7e-7, 8.0e-7 (largest 1.4e-6) in 4.83 /
// 4.54 / 4.48.  Workgroups without a live ray end at once, but with feature gradients one or two fit a CU, so
// that 65536 of them take 0.15 ms.  A head (FP16 records, 40 knots) in the middle of three 700 x 500 views of
// 11 voxels a pixel, plain: 0.22 ms, with the parts chosen by all the tiles 1.47.
static uint32_t bwd_parts(const KLaunch &L, const RaySplit &s, double hit)
{
    const double blocks = (double)tile_groups(L.W, L.H, L.ncam, 1, L.spread), live = blocks * hit;
    const double most = L.dfeat ? 16384.0 : 65536.0;  // live or not
    uint32_t parts = 1;
    while (parts < (uint32_t)s.lanes && blocks * parts * 2.0 <= most &&
           live * parts * 2.0 <= (parts == 1 ? 4096.0 : 1024.0))
        parts *= 2;
    return parts;
}

static hipError_t launch_any(const RenderArgs &a, hipStream_t st, int mode)
{
    for (int c0 = 0; c0 < a.ncam; c0 += kCamChunk) {
        KLaunch L = a.launch;
        L.ncam = a.ncam - c0 < kCamChunk ? a.ncam - c0 : kCamChunk;
        L.cam_base = c0;
        for (int i = 0; i < L.ncam; ++i) L.cams[i] = a.cams[c0 + i];
        ViewGeo geo = {0.0, 0.0, 0.0};
        for (int i = 0; i < L.ncam; ++i) {
            const ViewGeo v = view_geo(L.cams[i], L.W, L.H, a.grid);
            geo.pitch = fmax(geo.pitch, v.pitch);
            geo.chord = fmax(geo.chord, v.chord);
            geo.hit += v.hit / L.ncam;
        }
        const double rays = (double)L.W * L.H * L.ncam;
        const int want = mode == kBwd ? bwd_lanes(L, geo.pitch)
                                      : (mode == kFwd ? fwd_lanes(rays, a.feat.layout, a.feat.dtype, a.tf.K, geo) : 1);
        RaySplit split = fit_split({want, L.ncam % 8 != 0 ? 1u : 0u}, L.W, L.H, L.ncam, mode == kBwd);
        L.spread = split.spread;
        if (mode == kBwd) split.parts = bwd_parts(L, split, geo.hit);
        hipError_t e;
        const int lay = a.feat.layout, dt = a.feat.dtype;
        if (lay == DVR_PLANAR && dt == DVR_F32) e = launch_k<DVR_PLANAR, DVR_F32>(a.feat, a.grid, a.tf, a.rp, L, st, mode, split);
        else if (lay == DVR_PLANAR && dt == DVR_F16) e = launch_k<DVR_PLANAR, DVR_F16>(a.feat, a.grid, a.tf, a.rp, L, st, mode, split);
        else if (lay == DVR_INTERLEAVED && dt == DVR_F32) e = launch_k<DVR_INTERLEAVED, DVR_F32>(a.feat, a.grid, a.tf, a.rp, L, st, mode, split);
        else if (lay == DVR_INTERLEAVED && dt == DVR_F16) e = launch_k<DVR_INTERLEAVED, DVR_F16>(a.feat, a.grid, a.tf, a.rp, L, st, mode, split);
        else if (lay == DVR_SPLIT && dt == DVR_F32) e = launch_k<DVR_SPLIT, DVR_F32>(a.feat, a.grid, a.tf, a.rp, L, st, mode, split);
        else if (lay == DVR_SPLIT && dt == DVR_F16) e = launch_k<DVR_SPLIT, DVR_F16>(a.feat, a.grid, a.tf, a.rp, L, st, mode, split);
        else if (lay == DVR_QUAD && dt == DVR_F32) e = launch_k<DVR_QUAD, DVR_F32>(a.feat, a.grid, a.tf, a.rp, L, st, mode, split);
        else if (lay == DVR_QUAD && dt == DVR_F16) e = launch_k<DVR_QUAD, DVR_F16>(a.feat, a.grid, a.tf, a.rp, L, st, mode, split);
        else e = hipErrorInvalidValue;
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Empty-brick bits for one TF: brick i is empty when brick_empty() holds for its (min, max); a wave
// covers 64 bricks and writes the two 32-bit words of its ballot.
__global__ __launch_bounds__(256) void k_brick_mask(const float *__restrict__ bricks, int nb, KTF tf)
{
    __shared__ TFShared<64> sh;
    float kx[64];
    tf_load<64>(sh, kx, tf);
    __syncthreads();
    const int i = (int)(blockIdx.x * 256u + threadIdx.x);
    bool e = false;
    if (i < nb) e = brick_empty<64>(sh, kx, bricks[2 * i], bricks[2 * i + 1]);
    const uint64_t bal = __ballot(e);
    const int w0 = (int)(blockIdx.x * 256u + (threadIdx.x & ~63u)) / 32;  // first word of this wave
    const int nw = (nb + 31) / 32;
    uint32_t *mask = reinterpret_cast<uint32_t *>(const_cast<float *>(bricks) + 2 * nb);
    const int lane = threadIdx.x & 63;
    if (lane == 0 && w0 < nw) mask[w0] = (uint32_t)bal;
    if (lane == 1 && w0 + 1 < nw) mask[w0 + 1] = (uint32_t)(bal >> 32);
}

hipError_t launch_brick_mask(const RenderArgs &a, hipStream_t st)
{
    const int nb = a.feat.nb[0] * a.feat.nb[1] * a.feat.nb[2];
    hipLaunchKernelGGL(k_brick_mask, dim3((nb + 255) / 256), dim3(256), 0, st, a.feat.bricks, nb, a.tf);
    return hipGetLastError();
}

hipError_t launch_render(const RenderArgs &a, hipStream_t st)
{
    if (a.feat.bricks) {
        const hipError_t e = launch_brick_mask(a, st);
        if (e != hipSuccess) return e;
    }
    return launch_any(a, st, kFwd);
}
hipError_t launch_render_backward(const RenderArgs &a, hipStream_t st) { return launch_any(a, st, kBwd); }
hipError_t launch_render_gather(const RenderArgs &a, hipStream_t st)
{
    if (a.feat.bricks) {
        const hipError_t e = launch_brick_mask(a, st);
        if (e != hipSuccess) return e;
    }
    return launch_any(a, st, kGather);
}

}  // namespace dvr

namespace dvr {

__global__ __launch_bounds__(256) void k_fill_zero(float *p, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0.f;
}

hipError_t launch_fill_zero(float *p, int64_t n, hipStream_t st)
{
    const int64_t b = (n + 255) / 256;
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096)), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

}  // namespace dvr
