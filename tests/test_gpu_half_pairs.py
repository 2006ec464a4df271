"""FP16 planes read two voxels a load: rows of odd and even length put the pairs on every 2-byte boundary,
up to the last two voxels of an array.  The values are FP16-exact, so the same render from FP32 planes that
hold them does the same FP32 arithmetic: bits may differ only by how a product and a sum are contracted,
so the images agree to 2e-6 (values of order 1, a few tens of samples of 2^-24 each) and the ray state to
the sample."""
import numpy as np
import pytest
import torch

import paper_2605_19737_amd as dvr
import phantoms
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [abi.DVR_PLANAR, abi.DVR_SPLIT])
@pytest.mark.parametrize("shape", [(5, 7, 5), (4, 6, 8), (9, 5, 33), (3, 13, 14)])
@pytest.mark.parametrize("size", [(1100, 1100), (75, 62)])
def test_half_planes_equal_float_planes(layout, shape, size):
    rng = np.random.default_rng(11)
    w = phantoms.c4_volume(0, 64, 64)
    sp = (1.0, 0.9, 1.2)
    v16 = to_dev(rng.random(shape, dtype=np.float32), torch.float16)
    f16 = dvr.alloc_features(shape, sp, torch.float16, layout, bricks=False)
    dvr.features(v16, sp, [1.0], c=w.c, dtype=torch.float16, layout=layout, out=f16)
    f32 = dvr.alloc_features(shape, sp, torch.float32, layout, bricks=False)
    for name in ("grad", "kappa", "ves", "gmax"):
        if getattr(f16, name) is not None:
            getattr(f32, name).copy_(getattr(f16, name))
    ext = [h * (n - 1) for h, n in zip(sp, shape[::-1])]
    cam = abi.Camera()
    cam.persp, (cam.width, cam.height) = 0, size
    cam.d0[2] = 1.0
    cam.o[2] = -2.0
    cam.du[0], cam.dv[1] = ext[0] / size[0], ext[1] / size[1]  # up to the faces: the last cells are sampled
    params = dict(w.params, et_alpha=0.0)
    knots, rgba = to_dev(w.tf_knots), to_dev(w.tf_rgba)
    a = dvr.render(v16, f16, knots, rgba, params, [cam])
    b = dvr.render(v16.float(), f32, knots, rgba, params, [cam])
    assert torch.equal(a[2], b[2]) and int((a[2] >= 0).sum()) == size[0] * size[1]
    assert float(a[0].abs().max()) > 1e-3
    for x, y in zip(a[:2], b[:2]):
        assert float((x - y).abs().max()) <= 2e-6
