"""Batched launch with views that take different numbers of lanes per ray: images of odd sizes whose tile
tables end in padding, one view fine enough for one lane a ray beside coarse ones (4 lanes), and few rays
in all (16 lanes), on more volumes than the graph has feature branches.  A lane count changes which lane
computes a sample and not its arithmetic, so images and ray state equal the standalone calls bitwise."""
import numpy as np
import pytest
import torch

import paper_2605_19737_amd as dvr
import phantoms
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout,dtype", [(abi.DVR_QUAD, torch.float16), (abi.DVR_SPLIT, torch.float32),
                                          (abi.DVR_PLANAR, torch.float16)])
@pytest.mark.parametrize("sizes", [((1201, 1013), (131, 67)), ((37, 21), (1, 1), (64, 3))])
def test_batch_lane_counts_equal_standalone(layout, dtype, sizes):
    rng = np.random.default_rng(5)
    w = phantoms.c4_volume(0, 64, 64)
    shapes = [(19, 33, 41), (7, 30, 64), (24, 9, 17), (5, 48, 20), (12, 12, 70), (31, 21, 11)]
    sp = (0.7, 0.8, 1.9)
    vols = [to_dev(rng.random(s, dtype=np.float32), dtype) for s in shapes]
    feats = [dvr.alloc_features(s, sp, dtype, layout) for s in shapes]
    knots, rgba = to_dev(w.tf_knots), to_dev(w.tf_rgba)
    views = []
    for i, s in enumerate(shapes):
        ext = [h * (n - 1) for h, n in zip(sp, s[::-1])]
        for j, (W, H) in enumerate(sizes if i == 0 else sizes[-1:]):
            d0 = (0.3, 0.2 - 0.1 * j, 1.0)
            nrm = float(np.linalg.norm(d0))
            d0 = tuple(x / nrm for x in d0)
            cam = abi.Camera()
            cam.persp, cam.width, cam.height = 0, W, H
            for a in range(3):
                cam.d0[a] = d0[a]
                cam.o[a] = -2.0 * d0[a] * ext[2] if a == 2 else -0.1 * ext[a]
                cam.du[a] = 1.2 * ext[0] / W if a == 0 else 0.0
                cam.dv[a] = 1.2 * ext[1] / H if a == 1 else 0.0
            views.append((i, cam, torch.empty((H, W, 4), dtype=torch.float32, device="cuda"),
                          torch.empty((H, W), dtype=torch.float32, device="cuda"),
                          torch.empty((H, W), dtype=torch.int32, device="cuda")))
    b = dvr.Batch(vols, [sp] * len(vols), feats, views, [1.0], knots, rgba, w.params, c=w.c)
    for rep in range(2):
        for v in views:
            v[2].fill_(-1.0)
        b.launch()
        b.check()
        torch.cuda.synchronize()
        shaded = 0
        for i, cam, img, T, k in views:
            f = dvr.features(vols[i], sp, [1.0], c=w.c, dtype=dtype, layout=layout)
            assert torch.equal(f.grad, feats[i].grad) and torch.equal(f.gmax, feats[i].gmax)
            rimg, rT, rk = dvr.render(vols[i], f, knots, rgba, w.params, [cam])
            assert torch.equal(img, rimg[0]) and torch.equal(T, rT[0]) and torch.equal(k, rk[0])
            shaded += int((k >= 0).sum())
        assert shaded > 0
    b.close()
