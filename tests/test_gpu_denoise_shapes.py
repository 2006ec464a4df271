"""The denoise pre-pass on volumes far from a cube: rows so many that they exceed the workgroups a grid has
along y, and rows of a few voxels, which must not leave most of a wave idle.  The median against scipy's with clamped indices, bit for bit; the Gaussian against the FP64 oracle
(FP32 within 1e-6 of the range, as on the other shapes)."""
import numpy as np
import pytest
import torch
from scipy import ndimage

import oracle.denoise as od
import paper_2605_19737_amd as dvr
from tests.gpu_common import f32, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2, 300001, 2), (2, 530000, 3)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_median_of_many_rows(shape, dtype):
    print(f"[denoise shapes] median {shape} {dtype}", flush=True)
    v = to_dev(np.random.default_rng(shape[1]).random(shape, dtype=np.float32), dtype)
    got = dvr.denoise(v, (1.0, 1.0, 1.0)).float().cpu().numpy()
    np.testing.assert_array_equal(got, ndimage.median_filter(v.float().cpu().numpy(), size=3, mode="nearest"))


@pytest.mark.parametrize("shape", [(19, 37, 5), (7, 130, 17), (40, 67, 33), (3, 1000, 8), (18, 9, 2), (5, 70, 32)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_median_of_short_rows(shape, dtype):
    v = to_dev(np.random.default_rng(shape[1]).random(shape, dtype=np.float32), dtype)
    got = dvr.denoise(v, (1.0, 1.0, 1.0)).float().cpu().numpy()
    np.testing.assert_array_equal(got, ndimage.median_filter(v.float().cpu().numpy(), size=3, mode="nearest"))


def _us(f):
    f()
    best = float("inf")
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(20):
            f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 50.0)
    return best


@pytest.mark.parametrize("nx", [2, 8])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_median_of_short_rows_is_not_slow(nx, dtype):
    """A volume costs the same kind of time whichever axis is short (64 lanes on rows of 2 and 8 voxels made
    it six times as slow)."""
    t = []
    for shape in ((512, 512, nx), (nx, 512, 512)):
        v = torch.rand(shape, device="cuda").to(dtype)
        out = torch.empty_like(v)
        t.append(_us(lambda: dvr.denoise(v, (1.0, 1.0, 1.0), out=out)))
    print(f"[denoise shapes] median, short x {t[0]:.1f} us, short z {t[1]:.1f} us", flush=True)
    assert t[0] <= 3.0 * t[1]


def test_gauss_of_many_rows():
    shape, sigma = (2, 1100001, 2), f32(0.3)
    print(f"[denoise shapes] gauss {shape}", flush=True)
    v = to_dev(np.random.default_rng(1).random(shape, dtype=np.float32))
    got = dvr.denoise(v, (1.0, 1.0, 1.0), "gauss", sigma).cpu().numpy().astype(np.float64)
    ref = od.gauss(v.cpu().numpy(), (1.0, 1.0, 1.0), sigma)
    assert rel_err(got, ref) <= 1e-6


@pytest.mark.parametrize("sigma", [1.0, 2.0])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_gauss_of_short_rows_is_not_slow(sigma, dtype):
    """As for the median: tiles of 64 x 16 on rows of 8 voxels made it up to four times as slow."""
    t = []
    for shape in ((512, 512, 8), (8, 512, 512)):
        v = torch.rand(shape, device="cuda").to(dtype)
        out = torch.empty_like(v)
        t.append(_us(lambda: dvr.denoise(v, (1.0, 1.0, 1.0), "gauss", sigma, out=out)))
    print(f"[denoise shapes] gauss {sigma}, short x {t[0]:.1f} us, short z {t[1]:.1f} us", flush=True)
    assert t[0] <= 1.5 * t[1]
