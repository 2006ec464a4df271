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
