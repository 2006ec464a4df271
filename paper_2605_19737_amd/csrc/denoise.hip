// Optional denoise pre-pass (Sec. 5.3: lightweight spatial smoothing or median filtering as an
// optional compute pass before the morphology pass).
//   k_median3   3x3x3 median, clamp-to-edge: the neighbours are sorted along x, y and z in turn, which
//               leaves 19 candidates in a known partial order, and a pruned network selects the median.
//               Where a NaN is met: forgetful selection (keep 15, then repeatedly move the smallest and
//               the largest of the kept values to the ends, drop both and take in the next neighbour;
//               the median of the last three is the answer).  All indices are compile-time, so the
//               values stay in registers.  The result is one of the inputs (exact).
//   k_gauss     the separable sampled, normalized Gaussian (radius floor(3 sigma/h + 1/2), clamp-to-edge),
//               FP32 accumulation, in one pass: radii up to 8 on volumes of enough tiles.
//   k_smooth    one axis of it; three launches (x, y, z) through FP32 workspaces.
#include <type_traits>

#include "common.hpp"

namespace dvr {

template <int DT>
__device__ __forceinline__ float ld_any(const void *p, uint32_t i)
{
    if constexpr (DT == DVR_F32) return reinterpret_cast<const float *>(p)[i];
    else return __half2float(reinterpret_cast<const __half *>(p)[i]);
}

template <int DT>
__device__ __forceinline__ void st_any(void *p, uint32_t i, float v)
{
    if constexpr (DT == DVR_F32) reinterpret_cast<float *>(p)[i] = v;
    else reinterpret_cast<__half *>(p)[i] = __float2half_rn(v);
}

__device__ __forceinline__ void cswap(float &a, float &b)
{
    const float lo = fminf(a, b), hi = fmaxf(a, b);
    a = lo;
    b = hi;
}

// After this, b[0] is the smallest and b[N-1] the largest of b[0..N-1].
template <int N>
__device__ __forceinline__ void min_max_to_ends(float (&b)[15])
{
#pragma unroll
    for (int i = 0; i < N - 1; ++i) cswap(b[i], b[i + 1]);  // largest to N-1
#pragma unroll
    for (int i = N - 3; i >= 0; --i) cswap(b[i], b[i + 1]);  // smallest of 0..N-2 to 0
}

// one forgetful-selection step on a kept set of N values: drop the ends, take in x
template <int N>
__device__ __forceinline__ void forget_step(float (&b)[15], float x)
{
    min_max_to_ends<N>(b);
#pragma unroll
    for (int i = 0; i < N - 2; ++i) b[i] = b[i + 1];
    b[N - 2] = x;
}

// One voxel's median by forgetful selection (exact; a NaN among the 27 drops out of each comparison).
template <int DT>
__device__ __forceinline__ float median27(const void *__restrict__ in, int x, int y, int z, int nx, int ny, int nz)
{
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    float v[27];
#pragma unroll
    for (int k = 0; k < 27; ++k) {
        const int dz = k / 9 - 1, dy = (k / 3) % 3 - 1, dx = k % 3 - 1;
        const int zz = min(max(z + dz, 0), nz - 1), yy = min(max(y + dy, 0), ny - 1), xx = min(max(x + dx, 0), nx - 1);
        v[k] = ld_any<DT>(in, (uint32_t)zz * plane + (uint32_t)yy * nx + xx);
    }
    float b[15];
#pragma unroll
    for (int i = 0; i < 15; ++i) b[i] = v[i];
    forget_step<15>(b, v[15]);
    forget_step<14>(b, v[16]);
    forget_step<13>(b, v[17]);
    forget_step<12>(b, v[18]);
    forget_step<11>(b, v[19]);
    forget_step<10>(b, v[20]);
    forget_step<9>(b, v[21]);
    forget_step<8>(b, v[22]);
    forget_step<7>(b, v[23]);
    forget_step<6>(b, v[24]);
    forget_step<5>(b, v[25]);
    forget_step<4>(b, v[26]);
    // three left: their median
    return fmaxf(fminf(b[0], b[1]), fminf(fmaxf(b[0], b[1]), b[2]));
}

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float vmin(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ float vmax(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ h2 vmin(h2 a, h2 b) { return __builtin_elementwise_min(a, b); }
__device__ __forceinline__ h2 vmax(h2 a, h2 b) { return __builtin_elementwise_max(a, b); }

// a <= b <= c afterwards (without NaN)
__device__ __forceinline__ void sort3(float &a, float &b, float &c)
{
    const float lo = fminf(fminf(a, b), c), mid = __builtin_amdgcn_fmed3f(a, b, c), hi = fmaxf(fmaxf(a, b), c);
    a = lo;
    b = mid;
    c = hi;
}
__device__ __forceinline__ void sort3(h2 &a, h2 &b, h2 &c)
{
    const h2 t0 = vmin(a, b), t1 = vmax(a, b), t2 = vmin(t1, c);
    c = vmax(t1, c);
    a = vmin(t0, t2);
    b = vmax(t0, t2);
}

// Median of the 27 values m[9 i + 3 j + k] sorted along i, j and k: the eight corner-most (rank products
// above 14 from either end) cannot be it, and 44 comparators (70 minima and maxima) select the tenth of
// the other 19.  Every 0-1 input with that order (980 of them) comes out right, so every input does.
template <typename V>
__device__ __forceinline__ V median_cube(V (&m)[27])
{
    auto ce = [&](int a, int b) {
        const V lo = vmin(m[a], m[b]);
        m[b] = vmax(m[a], m[b]);
        m[a] = lo;
    };
    auto mn = [&](int a, int b) { m[a] = vmin(m[a], m[b]); };  // m[b] is not used again
    auto mx = [&](int a, int b) { m[b] = vmax(m[a], m[b]); };  // m[a] is not used again
    ce(10, 4); ce(8, 24); ce(5, 15); ce(14, 16); mx(12, 10); ce(6, 2); ce(7, 11); ce(8, 20); ce(14, 15); ce(4, 10);
    ce(7, 2); ce(21, 19); mn(24, 20); mx(6, 18); ce(7, 21); ce(2, 19); ce(11, 22); ce(10, 5); ce(13, 14); ce(2, 18);
    ce(11, 21); mx(4, 10); ce(13, 5); mx(7, 2); ce(11, 18); ce(21, 19); mx(10, 2); mx(13, 11); ce(5, 18); ce(14, 21);
    mn(15, 19); mn(16, 22); mx(2, 5); ce(11, 14); ce(15, 18); mn(16, 21); mx(11, 5); ce(14, 15); mx(16, 18); mx(5, 8);
    mn(14, 24); mn(18, 8); mn(15, 18); mn(14, 15);
    return m[14];
}

// Voxels per lane along y: 2 in FP16 (packed in one register), 1 in FP32.
template <int DT>
struct Med {
    using V = float;
    static constexpr int kY = 1;
};
template <>
struct Med<DVR_F16> {
    using V = h2;
    static constexpr int kY = 2;
};

// The 3 x 3 (x, y) neighbours of the lane's voxels in slice z (clamped), sorted along x and then y; nan:
// whether one of them is a NaN.
template <int DT>
__device__ __forceinline__ void med_slice(const void *__restrict__ in, const uint32_t (&row)[Med<DT>::kY + 2],
                                          const int (&col)[3], uint32_t base, typename Med<DT>::V (&s)[3][3], bool &nan)
{
    typename Med<DT>::V v[3][3];  // [y][x]
    if constexpr (DT == DVR_F32) {
        const float *p = reinterpret_cast<const float *>(in) + base;
#pragma unroll
        for (int y = 0; y < 3; ++y)
#pragma unroll
            for (int x = 0; x < 3; ++x) v[y][x] = p[row[y] + col[x]];
        nan = __builtin_isunordered(v[2][2], v[2][2]);
#pragma unroll
        for (int y = 0; y < 3; ++y) nan = nan || __builtin_isunordered(v[y][0], v[y][1]);
        nan = nan || __builtin_isunordered(v[0][2], v[1][2]);
    } else {
        const _Float16 *p = reinterpret_cast<const _Float16 *>(in) + base;
        _Float16 e[4][3];
        nan = false;
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int x = 0; x < 3; ++x) e[y][x] = p[row[y] + col[x]];
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            nan = nan || __builtin_isunordered(e[0][x], e[1][x]) || __builtin_isunordered(e[2][x], e[3][x]);
#pragma unroll
            for (int y = 0; y < 3; ++y) v[y][x] = h2{e[y][x], e[y + 1][x]};
        }
    }
#pragma unroll
    for (int y = 0; y < 3; ++y) sort3(v[y][0], v[y][1], v[y][2]);
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        sort3(v[0][x], v[1][x], v[2][x]);
#pragma unroll
        for (int y = 0; y < 3; ++y) s[y][x] = v[y][x];
    }
}

// A wave takes 64 consecutive voxels of x, or on rows of at most 32 voxels 1 << lw columns of 64 >> lw groups
// of rows (8 x 512 x 512: FP32 68 -> 13 us, FP16 78 -> 13; one lane a voxel with 27 loads took 29 and 28); a lane walks a run of z, sorting each slice's 3 x 3
// neighbours once for the three voxels that share them.  Bound by VALU issue: per voxel 107 minimum and
// maximum instructions in FP32 and 77 in FP16 (two voxels an instruction) against 388 for a selection
// from 27 unsorted values: 512 x 512 x 400 FP16 1.30 -> 0.37 ms, FP32 1.30 -> 0.44.  The waves that meet a NaN take that
// selection instead (median27), whose answer then depends on its own order of comparisons.
template <int DT>
__global__ __launch_bounds__(256) void k_median3(const void *__restrict__ in, void *__restrict__ out, int nx, int ny,
                                                 int nz, int run, int lw, unsigned by0)
{
    using V = typename Med<DT>::V;
    constexpr int kY = Med<DT>::kY;
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    const uint32_t lane = threadIdx.x & 63u;
    const int x = (int)((blockIdx.x << lw) + (lane & ((1u << lw) - 1u)));
    const int y0 = (int)((((by0 + blockIdx.y) * 4u + (threadIdx.x >> 6)) << (6 - lw)) + (lane >> lw)) * kY;
    if (x >= nx || y0 >= ny) return;
    const int z0 = (int)blockIdx.z * run, z1 = min(z0 + run, nz);
    uint32_t row[kY + 2];
#pragma unroll
    for (int r = 0; r < kY + 2; ++r) row[r] = (uint32_t)min(max(y0 - 1 + r, 0), ny - 1) * (uint32_t)nx;
    const int col[3] = {max(x - 1, 0), x, min(x + 1, nx - 1)};
    V a[3][3], b[3][3], c[3][3];  // slices z - 1, z, z + 1
    bool na, nb, nc;
    med_slice<DT>(in, row, col, (uint32_t)max(z0 - 1, 0) * plane, a, na);
    med_slice<DT>(in, row, col, (uint32_t)z0 * plane, b, nb);
#pragma unroll 3
    for (int z = z0; z < z1; ++z) {
        med_slice<DT>(in, row, col, (uint32_t)min(z + 1, nz - 1) * plane, c, nc);
        V m[27];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                m[9 * i + 3 * j] = a[i][j];
                m[9 * i + 3 * j + 1] = b[i][j];
                m[9 * i + 3 * j + 2] = c[i][j];
                sort3(m[9 * i + 3 * j], m[9 * i + 3 * j + 1], m[9 * i + 3 * j + 2]);
            }
        const V med = median_cube(m);
        const uint32_t o = (uint32_t)z * plane + (uint32_t)y0 * nx + x;
        if (!__any(na || nb || nc)) {
            if constexpr (DT == DVR_F32) {
                reinterpret_cast<float *>(out)[o] = med;
            } else {
                reinterpret_cast<_Float16 *>(out)[o] = med.x;
                if (y0 + 1 < ny) reinterpret_cast<_Float16 *>(out)[o + (uint32_t)nx] = med.y;
            }
        } else {
            for (int e = 0; e < kY && y0 + e < ny; ++e)
                st_any<DT>(out, o + (uint32_t)e * nx, median27<DT>(in, x, y0 + e, z, nx, ny, nz));
        }
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                a[i][j] = b[i][j];
                b[i][j] = c[i][j];
            }
        na = nb;
        nb = nc;
    }
}

template <int DT>
static void launch_median(const void *vol, const dvr_grid &g, void *out, hipStream_t st)
{
    int lw = 6;
    while (lw > 1 && (1 << (lw - 1)) >= g.nx) --lw;
    const int per = (256 >> lw) * Med<DT>::kY;
    const unsigned bx = (unsigned)((g.nx + (1 << lw) - 1) >> lw), by = (unsigned)((g.ny + per - 1) / per);
    // a run sorts run + 2 slices for run voxels; short runs where long ones would not fill the chip
    int run = 16;
    while (run > 1 && (int64_t)bx * by * ((g.nz + run - 1) / run) < 2048) run >>= 1;
    for (unsigned b = 0; b < by; b += kMaxGridYZ)
        hipLaunchKernelGGL(k_median3<DT>, dim3(bx, min(by - b, kMaxGridYZ), (unsigned)((g.nz + run - 1) / run)), dim3(256),
                           0, st, vol, out, g.nx, g.ny, g.nz, run, lw, b);
}

struct GaussTaps {
    int r;
    float w[DVR_MAX_RADIUS + 1];
};

// The three axes in one pass, radii up to P in the plane and RZ in z.  A workgroup walks a 64 x 16 tile
// along z: each slice (with halo, clamped to the edge, the next one's loads in flight) is staged, filtered
// along x into a second LDS array and along y into registers, where the last 2 RZ + 1 slices' values wait
// for the z filter.  The sums are k_smooth's, in its order, so the result is the same bits.  The
// volume is read and written once where three passes through FP32 workspaces moved 20 bytes a voxel.  No
// unit bounds it alone (512 x 512 x 400 FP16, radius 3: texture data busy on 77 % of the cycles, VALU issue
// 58 %, no bank conflicts): a slice is a chain of two barriers, loads and two filters, with 13 waves a SIMD
// over the whole launch.  P (the halo's room) makes every LDS offset a constant.
template <int DT, int P, int RZ>
__global__ __launch_bounds__(256) void k_gauss(const void *__restrict__ in, void *__restrict__ out, int nx, int ny, int nz,
                                               GaussTaps tx, GaussTaps ty, GaussTaps tz, int run)
{
    constexpr int TX = 64, TY = 16, W = TX + 2 * P, HH = TY + 2 * P, NR = (HH + 3) / 4;
    __shared__ float F[HH * W], M[HH * TX];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int x0 = (int)blockIdx.x * TX, y0 = (int)blockIdx.y * TY;
    const int z0 = (int)blockIdx.z * run, z1 = min(z0 + run, nz);
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    const int rx = tx.r, ry = ty.r;
    const int xm = min(x0 + lane, nx - 1);                              // this lane's column,
    const int hc = lane < rx ? P - rx + lane : P + TX + (lane - rx);    // and its halo column of the staged rows
    const int xh = min(max(x0 - P + hc, 0), nx - 1);
    using E = std::conditional_t<DT == DVR_F32, float, __half>;  // widened when stored: a conversion here would wait
    const E *src = reinterpret_cast<const E *>(in);
    E a[NR], h[NR];
    auto load = [&](int z) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int j = wv + 4 * i;
            if (j < P - ry || j >= P + TY + ry) continue;
            const uint32_t row = (uint32_t)z * plane + (uint32_t)min(max(y0 - P + j, 0), ny - 1) * (uint32_t)nx;
            a[i] = src[row + xm];
            if (lane < 2 * rx) h[i] = src[row + xh];
        }
    };
    float ring[4][2 * RZ + 1];
    load(max(z0 - RZ, 0));
    for (int s = z0 - RZ; s < z1 + RZ; ++s) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int k = 0; k < 2 * RZ; ++k) ring[i][k] = ring[i][k + 1];
        const int z = min(max(s, 0), nz - 1);
        if (s == z0 - RZ || (s > 0 && s < nz)) {  // else the clamped slice once more
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int j = wv + 4 * i;
                if (j < P - ry || j >= P + TY + ry) continue;
                F[j * W + P + lane] = ld_any<DT>(&a[i], 0);
                if (lane < 2 * rx) F[j * W + hc] = ld_any<DT>(&h[i], 0);
            }
            __syncthreads();  // F is staged, and M's readers of the slice before are done
            if (z + 1 < min(z1 + RZ, nz)) load(z + 1);
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int j = wv + 4 * i;
                if (j < P - ry || j >= P + TY + ry) continue;
                const float *f = F + j * W + lane;
                float acc = tx.w[0] * f[P];
#pragma unroll
                for (int m = 1; m <= P; ++m)
                    if (m <= rx) acc = fmaf(tx.w[m], f[P + m] + f[P - m], acc);
                M[j * TX + lane] = acc;
            }
            __syncthreads();  // M is there, and F's readers are done
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float *f = M + (wv * 4 + i) * TX + lane;
                float acc = ty.w[0] * f[P * TX];
#pragma unroll
                for (int m = 1; m <= P; ++m)
                    if (m <= ry) acc = fmaf(ty.w[m], f[(P + m) * TX] + f[(P - m) * TX], acc);
                ring[i][2 * RZ] = acc;
            }
        }
        if (s >= z0 + RZ) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float acc = tz.w[0] * ring[i][RZ];
#pragma unroll
                for (int m = 1; m <= RZ; ++m)
                    if (m <= tz.r) acc = fmaf(tz.w[m], ring[i][RZ + m] + ring[i][RZ - m], acc);
                const int y = y0 + wv * 4 + i;
                if (x0 + lane < nx && y < ny)
                    st_any<DT>(out, (uint32_t)(s - RZ) * plane + (uint32_t)y * (uint32_t)nx + x0 + lane, acc);
            }
        }
    }
}

// Slices per run of the one-pass Gaussian, 0 for three passes.  A run filters 2 RZ slices more than it
// writes and its slices follow each other (1.3-2 us each up to radius 4, 3.4-4.6 above), so long runs are for
// volumes that fill the chip with them, and one that cannot be cut into enough runs is left to the three
// passes.  us, radius 2 / 3 / 4 / 5 / 8 (FP16; FP32 is within 10 %): 512 x 512 x 400 (3328 workgroups at 32)
// 186 / 248 / 342 / 601 / 1111, three passes 1165 / 1360 / 1543 / 1711 / 2191; 400 x 300 x 100 (931 at 16)
// 46 / 59 / 71 / 119 / 277, 123 / 147 / 168 / 192 / 264; 220 x 200 x 180 (1196 at 8) 32 / 43 / 54, 74 / 89 /
// 104; 256 x 256 x 40 (640 at 4) 20 / 29 / 36, 34 / 39 / 44; 97 x 113 x 61 (256 at 4) 18 / 26 / 34, 18 / 20 / 22.
// Tiles filled to less than half (0.6 above radius 3) are left to the three passes too, radius 2 / 3 / 4 / 6:
// 8 x 512 x 512 (an eighth) 43 / 56 / 69 / 126, three passes 20 / 22 / 24 / 31; 20 x 512 x 512 (0.31) 43 / 57 /
// 70 / 126, 47 / 53 / 62 / 76; 512 x 8 x 512 (0.5) 19 / 27 / 35, 26 / 30 / 31; 66 x 300 x 300 (0.51) 32 / 43 /
// 83, 58 / 67 / 76; 40 x 300 x 300 (0.62) 26 / 35 / 45, 40 / 47 / 53.
static int gauss_run(const dvr_grid &g, int r)
{
    if (r > 8 || (unsigned)(g.ny + 15) / 16 > kMaxGridYZ) return 0;
    const int64_t tiles = (int64_t)((g.nx + 63) / 64) * ((g.ny + 15) / 16);
    if ((double)g.nx * g.ny < (r <= 3 ? 0.5 : 0.6) * 1024.0 * (double)tiles) return 0;
    auto groups = [&](int run) { return tiles * ((g.nz + run - 1) / run); };
    if (groups(32) >= 1536) return 32;
    if (groups(16) >= 900 && r <= 6) return 16;
    if (r > 4) return 0;
    return groups(8) >= 700 ? 8 : (groups(4) >= 600 ? 4 : 0);
}

template <int DT, int P>
static hipError_t launch_gauss(const void *vol, const dvr_grid &g, const GaussTaps (&t)[3], int run, void *out,
                               hipStream_t st)
{
    const unsigned bx = (unsigned)((g.nx + 63) / 64), by = (unsigned)((g.ny + 15) / 16);
    const dim3 grid(bx, by, (unsigned)((g.nz + run - 1) / run));
#define DVR_G(RZ)                                                                                                     \
    if (t[2].r <= RZ) {                                                                                               \
        hipLaunchKernelGGL((k_gauss<DT, P, RZ>), grid, dim3(256), 0, st, vol, out, g.nx, g.ny, g.nz, t[0], t[1], t[2], run); \
        return hipGetLastError();                                                                                     \
    }
    DVR_G(1)
    DVR_G(2)
    DVR_G(3)
    DVR_G(4)
    DVR_G(6)
    DVR_G(8)
#undef DVR_G
    return hipErrorInvalidValue;
}

// out = G_axis * in along one axis (stride in elements, n the axis length)
template <int DTI, int DTO>
__global__ __launch_bounds__(256) void k_smooth(const void *__restrict__ in, void *__restrict__ out, int nx, int ny,
                                                int nz, int axis, GaussTaps t)
{
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    const uint32_t e = blockIdx.x * 256u + threadIdx.x;
    if (e >= plane) return;
    const int z = (int)blockIdx.y;
    const int y = (int)(e / (uint32_t)nx), x = (int)(e - (uint32_t)y * nx);
    const int pos = axis == 0 ? x : (axis == 1 ? y : z);
    const int n = axis == 0 ? nx : (axis == 1 ? ny : nz);
    const uint32_t st = axis == 0 ? 1u : (axis == 1 ? (uint32_t)nx : plane);
    const uint32_t base = (uint32_t)z * plane + e - (uint32_t)pos * st;
    float acc = t.w[0] * ld_any<DTI>(in, base + (uint32_t)pos * st);
    for (int m = 1; m <= t.r; ++m) {
        const int a = min(pos + m, n - 1), b = max(pos - m, 0);
        acc = fmaf(t.w[m], ld_any<DTI>(in, base + (uint32_t)a * st) + ld_any<DTI>(in, base + (uint32_t)b * st), acc);
    }
    st_any<DTO>(out, (uint32_t)z * plane + e, acc);
}

hipError_t launch_denoise(const void *vol, int dt, const dvr_grid &g, int mode, const int r[3],
                          const float w[3][DVR_MAX_RADIUS + 1], void *out, float *ws, hipStream_t st)
{
    const uint32_t plane = (uint32_t)g.nx * (uint32_t)g.ny;
    const dim3 grid((plane + 255) / 256, g.nz);
    if (mode == DVR_DENOISE_MEDIAN3) {
        if (dt == DVR_F32) launch_median<DVR_F32>(vol, g, out, st);
        else launch_median<DVR_F16>(vol, g, out, st);
        return hipGetLastError();
    }
    GaussTaps t[3];
    for (int a = 0; a < 3; ++a) {
        t[a].r = r[a];
        for (int j = 0; j <= DVR_MAX_RADIUS; ++j) t[a].w[j] = w[a][j];
    }
    if (const int run = gauss_run(g, max(t[0].r, max(t[1].r, t[2].r)))) {
        if (t[0].r <= 4 && t[1].r <= 4)
            return dt == DVR_F32 ? launch_gauss<DVR_F32, 4>(vol, g, t, run, out, st)
                                 : launch_gauss<DVR_F16, 4>(vol, g, t, run, out, st);
        return dt == DVR_F32 ? launch_gauss<DVR_F32, 8>(vol, g, t, run, out, st)
                             : launch_gauss<DVR_F16, 8>(vol, g, t, run, out, st);
    }
    // one axis a launch
    const size_t N = (size_t)plane * g.nz;
    float *w0 = ws, *w1 = ws + N;
    if (dt == DVR_F32)
        hipLaunchKernelGGL((k_smooth<DVR_F32, DVR_F32>), grid, dim3(256), 0, st, vol, w0, g.nx, g.ny, g.nz, 0, t[0]);
    else
        hipLaunchKernelGGL((k_smooth<DVR_F16, DVR_F32>), grid, dim3(256), 0, st, vol, w0, g.nx, g.ny, g.nz, 0, t[0]);
    hipLaunchKernelGGL((k_smooth<DVR_F32, DVR_F32>), grid, dim3(256), 0, st, w0, w1, g.nx, g.ny, g.nz, 1, t[1]);
    if (dt == DVR_F32)
        hipLaunchKernelGGL((k_smooth<DVR_F32, DVR_F32>), grid, dim3(256), 0, st, w1, out, g.nx, g.ny, g.nz, 2, t[2]);
    else
        hipLaunchKernelGGL((k_smooth<DVR_F32, DVR_F16>), grid, dim3(256), 0, st, w1, out, g.nx, g.ny, g.nz, 2, t[2]);
    return hipGetLastError();
}

}  // namespace dvr
