"""The 3x3x3 median at the edges of its tiles (64 voxels of x per wave, 2 of y per lane in FP16, runs of z)
against scipy's median filter with clamped indices: bit-exact, infinities included; and next to a NaN,
where every window without one keeps its exact median."""
import numpy as np
import pytest
import torch
from scipy import ndimage

import paper_2605_19737_amd as dvr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(2, 2, 2), (64, 8, 16), (65, 9, 17), (63, 7, 33), (130, 5, 3), (3, 131, 2), (1 + 256, 2, 40)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_median_edges(dims, dtype):
    nx, ny, nz = dims
    rng = np.random.default_rng(nx * 1000 + ny * 10 + nz)
    v = torch.from_numpy(rng.standard_normal((nz, ny, nx)).astype(np.float32)).to(dtype)
    v.view(-1)[rng.integers(0, v.numel(), 3)] = float("inf")
    v.view(-1)[rng.integers(0, v.numel(), 3)] = -float("inf")
    v.view(-1)[rng.integers(0, v.numel(), v.numel() // 4)] = 0.5  # ties
    print(f"[median] {dims} {dtype}", flush=True)
    got = dvr.denoise(v.cuda(), (1.0, 1.0, 1.0)).cpu()
    ref = ndimage.median_filter(v.float().numpy(), size=3, mode="nearest")
    np.testing.assert_array_equal(got.float().numpy(), ref)
    # one NaN in the middle: its 3 x 3 x 3 neighbourhood may take any of its values, the rest is unchanged
    w = v.clone()
    c = (nz // 2, ny // 2, nx // 2)
    w[c] = float("nan")
    near = np.zeros(v.shape, bool)
    near[tuple(slice(max(i - 1, 0), i + 2) for i in c)] = True
    got = dvr.denoise(w.cuda(), (1.0, 1.0, 1.0)).cpu().float().numpy()
    np.testing.assert_array_equal(got[~near], ref[~near])
