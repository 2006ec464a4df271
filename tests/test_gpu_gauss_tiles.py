"""The Gaussian pre-pass at the edges of its 64 x 16 tiles and its runs of slices, for the
reaches it is built for (radii 1-8) and reaches that differ by axis, against the
FP64 oracle: FP32 within 1e-6 of the range (three sums of at most 19 terms of weight sum 1), FP16 within
one unit of the rounded FP64 value."""
import numpy as np
import pytest
import torch

import oracle.denoise as od
import paper_2605_19737_amd as dvr
from tests.gpu_common import rel_err, to_dev

pytestmark = pytest.mark.gpu

# 4, 8, 16 and 32 slices a run (each with remainders in x, y and z), and shapes left to the three passes
CASES = [((2, 2, 2), (1.0, 1.0, 1.0), 0.3), ((5, 16, 64), (1.0, 1.0, 1.0), 0.6), ((131, 193, 65), (1.0, 1.0, 1.0), 0.3),
         ((97, 145, 130), (1.0, 1.0, 1.0), 0.6), ((101, 129, 257), (1.0, 1.0, 1.0), 1.0),
         ((98, 255, 257), (0.8, 1.0, 2.0), 1.0), ((70, 400, 385), (1.0, 1.1, 1.0), 1.3),
         ((2, 1201, 1300), (1.0, 1.0, 0.3), 0.7), ((3, 1201, 1300), (1.0, 1.0, 0.6), 1.0),
         ((129, 257, 400), (1.0, 1.0, 1.0), 1.7), ((35, 1000, 450), (1.0, 1.0, 1.0), 2.0),
         ((33, 780, 1000), (1.0, 3.0, 0.9), 2.3), ((12, 31, 66), (1.0, 3.0, 0.4), 0.9), ((6, 18, 30), (1.0, 1.0, 1.0), 3.0)]


@pytest.mark.parametrize("shape,spacing,sigma", CASES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_gauss_tiles(shape, spacing, sigma, dtype):
    rng = np.random.default_rng(sum(shape))
    v = to_dev(rng.random(shape).astype(np.float32), dtype)
    out = torch.full_like(v, float("nan"))
    got = dvr.denoise(v, spacing, "gauss", sigma, out=out).float().cpu().numpy().astype(np.float64)
    ref = od.gauss(v.float().cpu().numpy(), tuple(float(np.float32(h)) for h in spacing), float(np.float32(sigma)))
    if dtype == torch.float32:
        assert rel_err(got, ref) <= 1e-6
    else:
        r16 = ref.astype(np.float16).astype(np.float64)
        assert np.all(np.abs(got - r16) <= np.spacing(np.abs(r16).astype(np.float16)).astype(np.float64))
