"""The denoise pre-pass on volumes far from a cube: rows so many that they exceed the workgroups a grid has
along y.  The median against scipy's with clamped indices, bit for bit; the Gaussian against the FP64 oracle
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


def test_gauss_of_many_rows():
    shape, sigma = (2, 1100001, 2), f32(0.3)
    print(f"[denoise shapes] gauss {shape}", flush=True)
    v = to_dev(np.random.default_rng(1).random(shape, dtype=np.float32))
    got = dvr.denoise(v, (1.0, 1.0, 1.0), "gauss", sigma).cpu().numpy().astype(np.float64)
    ref = od.gauss(v.cpu().numpy(), (1.0, 1.0, 1.0), sigma)
    assert rel_err(got, ref) <= 1e-6
