"""The split of a raymarch over lanes and workgroups (lanes.hpp) on the CPU: the rules are host code, so the
header is compiled into a small program.  Every launch the library accepts (up to 2^31 - 1 pixels, images up
to 2^23 on a side, 32 views a launch) must fit in one grid, of fewer than 2^32 threads, unless one lane per
ray on contiguous tiles does not fit either."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parents[1]
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

FIT = r"""
#include <cstdio>
#include "lanes.hpp"
using namespace dvr;
int main()
{
    long cases = 0, bad = 0, lost = 0, kept = 0;
    for (int lw = 0; lw <= 23; ++lw)
        for (int lh = 0; lh <= 23; ++lh)
            for (int odd = -1; odd <= 1; ++odd)
                for (int ncam = 1; ncam <= 32; ++ncam) {
                    const int W = (1 << lw) + (lw > 1 && lw < 23 ? odd : 0), H = (1 << lh) + (lh > 1 && lh < 23 ? odd : 0);
                    if ((double)W * H * ncam > 2147483647.0) continue;
                    for (int lanes = 1; lanes <= 16; lanes *= 4)
                        for (int adjoint = 0; adjoint < 2; ++adjoint) {
                            const uint32_t spread = ncam % 8 != 0;
                            const RaySplit s = fit_split({lanes, spread}, W, H, ncam, adjoint);
                            const int g = adjoint ? 1 : s.lanes;
                            const uint64_t n = tile_groups(W, H, ncam, g, s.spread);
                            const uint64_t tiles = (uint64_t)((W + 15) / 16) * ((H + 15) / 16) * ncam;
                            ++cases;
                            // every pixel has a workgroup, in whole rounds of the 8 XCDs
                            if (n % 8 || n * (256 / g) < (uint64_t)W * H * ncam) ++bad;
                            if (n * 256 >= (1ull << 32) && (tiles + 7) / 8 * 8 * 256 < (1ull << 32)) ++lost;
                            // nothing changes where the wanted split fits
                            if (tile_groups(W, H, ncam, adjoint ? 1 : lanes, spread) * 256 < (1ull << 32))
                                kept += s.lanes != lanes || s.spread != spread;
                        }
                }
    // 2^30 pixels at a coarse pitch: 4 lanes wanted, one fits
    const RaySplit s = fit_split({4, 1}, 32768, 32768, 1, false);
    printf("%ld %ld %ld %ld %d\n", cases, bad, lost, kept, s.lanes);
    return 0;
}
"""


def _run(tmp_path, src):
    (tmp_path / "t.cpp").write_text(src)
    exe = tmp_path / "t"
    subprocess.run([HIPCC, "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-O2", "-std=c++17", "-I", str(ROOT / "include"),
                    "-I", str(ROOT / "paper_2605_19737_amd" / "csrc"), "-I", "/opt/rocm/include", "-o", str(exe),
                    str(tmp_path / "t.cpp")], check=True, capture_output=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout


@pytest.mark.skipif(not Path(HIPCC).exists(), reason="needs hipcc")
def test_every_accepted_launch_fits_one_grid(tmp_path):
    cases, bad, lost, kept, lanes = map(int, _run(tmp_path, FIT).split())
    assert cases > 50000
    assert bad == 0 and lost == 0 and kept == 0 and lanes == 1


LANES = r"""
#include <cstdio>
#include "lanes.hpp"
using namespace dvr;
// an orthographic view along z of a box of nx x ny x nz voxels of h mm, `pitch` voxels a pixel, W x H pixels
static ViewGeo geo(int nx, int ny, int nz, float h, float pitch, int W, int H, float step)
{
    KGrid g;
    const float hh[3] = {h, h, h};
    g.n[0] = nx; g.n[1] = ny; g.n[2] = nz;
    set_grid_steps(g, hh, step);
    KCam c = {0, {0, 0, -100}, {0, 0, 1}, {pitch * h, 0, 0}, {0, pitch * h, 0}};
    return view_geo(c, W, H, g);
}
int main()
{
    const ViewGeo a = geo(41, 61, 101, 0.5f, 2.0f, 100, 60, 0.5f);
    printf("%.6f %.6f %.6f\n", a.pitch, a.chord, a.hit);
    KGrid g;
    const float hh[3] = {1, 1, 1};
    g.n[0] = g.n[1] = g.n[2] = 101;
    set_grid_steps(g, hh, 0.5f);
    // perspective from 200 mm before the box's centre: a pixel is 0.01 rad, 2 voxels there
    KCam c = {1, {50, 50, -150}, {-1, -1, 1}, {0.01f, 0, 0}, {0, 0.01f, 0}};
    const ViewGeo p = view_geo(c, 200, 200, g);
    printf("%.6f %.6f %.6f\n", p.pitch, p.chord, p.hit);
    // lanes: few rays; a dense coarse view; a fine one; thin and small volumes in large images
    printf("%d %d %d %d %d %d %d\n", fwd_lanes(16384, 3, 0, 8, geo(181, 217, 181, 1, 1.3f, 128, 128, 0.5f)),
           fwd_lanes(8388608, 2, 0, 4, geo(152, 229, 177, 1, 0.4f, 512, 512, 0.5f)),
           fwd_lanes(8388608, 2, 0, 4, geo(152, 229, 177, 1, 0.7f, 512, 512, 0.5f)),
           fwd_lanes(648000, 0, 0, 8, geo(152, 229, 177, 1, 3.8f, 180, 180, 0.5f)),
           fwd_lanes(6750000, 2, 0, 8, geo(231, 286, 6, 1, 1.47f, 1500, 1500, 0.5f)),
           fwd_lanes(1050000, 2, 0, 8, geo(231, 286, 6, 1, 4.7f, 700, 500, 0.5f)),
           fwd_lanes(37748736, 3, 0, 40, geo(181, 217, 181, 1, 2.5f, 2048, 2048, 0.5f)));
    return 0;
}
"""


@pytest.mark.skipif(not Path(HIPCC).exists(), reason="needs hipcc")
def test_lanes_follow_what_the_view_shows(tmp_path):
    o, p, lanes = _run(tmp_path, LANES).splitlines()
    # 40 x 60 x 100 steps of 0.5 mm seen along z: 50 mm of 0.25 mm samples over 20 x 30 mm of 100 x 60 mm
    assert [float(x) for x in o.split()] == pytest.approx([2.0, 200.0, 0.1], rel=1e-6)
    # 100 mm of 0.5 mm samples over 100^2 mm^2 of (200 x 2 mm)^2 at the centre
    assert [float(x) for x in p.split()] == pytest.approx([2.0, 200.0, 1.0 / 16.0], rel=1e-6)
    assert [int(x) for x in lanes.split()] == [16, 1, 4, 16, 1, 1, 1]


SCENE = r"""
#include <cstdio>
#include "lanes.hpp"
using namespace dvr;
int main()
{
    KGrid g;
    const float h[3] = {@H@};
    g.n[0] = @NX@; g.n[1] = @NY@; g.n[2] = @NZ@;
    const KCam cams[] = {@CAMS@};
    for (float step : {0.5f, 0.37f}) {
        set_grid_steps(g, h, step);
        for (int layout = 0; layout < 4; ++layout)
            for (int dtype = 0; dtype < 2; ++dtype)
                for (int n : {32, 8, 1})
                    for (int i = 0; i < 32; i += n) {
                        ViewGeo v = {0, 0, 0};
                        for (int k = i; k < i + n; ++k) {
                            const ViewGeo o = view_geo(cams[k], @W@, @HH@, g);
                            v.pitch = fmax(v.pitch, o.pitch);
                            v.chord = fmax(v.chord, o.chord);
                            v.hit += o.hit / n;
                        }
                        printf("%d %d\n", n, fwd_lanes((double)@W@ * @HH@ * n, layout, dtype, 8, v));
                    }
    }
    return 0;
}
"""


@pytest.mark.skipif(not Path(HIPCC).exists(), reason="needs hipcc")
@pytest.mark.parametrize("persp", [False, True])
def test_lanes_of_the_compared_launches(tmp_path, persp):
    """The launches of 32, 8 and 1 views that test_gpu_one_lane.py compares take 1, 4 and 16 lanes."""
    from tests import test_gpu_one_lane as t

    def vec(v):
        return "{" + ", ".join("%.9gf" % float(x) if "." in "%.9g" % float(x) or "e" in "%.9g" % float(x) else "%.1ff" % float(x)
                               for x in v) + "}"

    cams = ", ".join("{%d, %s, %s, %s, %s}" % (c.persp, vec(c.o), vec(c.d0), vec(c.du), vec(c.dv)) for c in t.cameras(persp))
    src = SCENE
    for key, val in dict(H=", ".join("%.1ff" % x for x in t.SP), NX=t.SHAPE[2], NY=t.SHAPE[1], NZ=t.SHAPE[0], CAMS=cams, W=t.W,
                         HH=t.H).items():
        src = src.replace("@%s@" % key, str(val))
    got = set(tuple(map(int, line.split())) for line in _run(tmp_path, src).splitlines())
    assert got == {(32, 1), (8, 4), (1, 16)}
