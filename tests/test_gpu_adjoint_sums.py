"""The sums that every workgroup of the render adjoint adds to, one FP32 word each: dL/d|g|_max and the TF
gradient, where a tile's rays are shared among workgroups.  Each add rounds the word (by up to half a unit of its
last place, 2.6e-8 of it rms on the average), n adds of one sign by 2.6e-8 sqrt(n / 3) of the sum, so there may
not be many more of them than with one lane per ray: about 1024, which is 4.8e-7, or 3.8e-7 on the mean of the
magnitudes.  That mean over twenty upstream gradients of different scale, against the FP64 oracle, stays within
1.6 times this for dL/d|g|_max (6e-7) and, normwise, within 1e-6 for the TF gradient, whose 1024 is an estimate
and whose samples' own rounding is added."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_19737_amd as dvr
import phantoms
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import f32, feats_np, oracle_params, sp32, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,side,views", [((200, 150, 180), 150, 6), ((150, 150, 150), 110, 10)])
def test_rounding_of_the_shared_sums(shape, side, views):
    h = (1.0, 1.0, 1.0)
    z, y, x = np.meshgrid(*[np.linspace(0, 1, n) for n in shape], indexing="ij")
    vol = (0.45 + 0.4 * np.sin(5 * x + 1) * np.cos(4 * y) * np.sin(3 * z + 0.5)).astype(np.float32)
    # 1.2 times the box's diagonal across, 2.5 and 2.8 voxels a pixel: 16 lanes per ray, about 200 tiles with live rays
    dims = shape[::-1]
    cams = [phantoms.ortho_camera(dims, h, 360.0 * v / views + 10.0, 20.0, side, side, span=1.2 * phantoms.box_diag(dims, h))
            for v in range(views)]
    knots = np.linspace(0.0, 1.0, 4).astype(np.float32)
    rgba = np.array([[0.2, 0.5, 0.8, 0.01], [0.3, 0.5, 1.0, 0.02], [0.9, 0.6, 0.5, 0.03], [0.9, 0.9, 0.8, 0.05]], np.float32)
    prm = phantoms.render_params(lambda_g=0.7, lambda_k=0.5, lambda_v=0.8, step_vox=1.0, et_alpha=0.0)
    dv = to_dev(vol)
    f = dvr.features(dv, h, [1.0], c=0.2, layout=abi.DVR_SPLIT).without_bricks()
    kn, tf = to_dev(knots), to_dev(rgba)
    img, T, k = dvr.render(dv, f, kn, tf, prm, cams)
    got = feats_np(f)
    rtf, _, rfg = oracle.render_vjp(vol.astype(np.float64), got, got["gmax"], sp32(h), knots, rgba, oracle_params(prm), cams,
                                    np.ones(tuple(img.shape), np.float32), want_features=True)
    e_max, e_tf = [], []
    for i in range(20):
        scale = f32(1.0 + 0.37 * i)  # the gradients are linear in it
        dtf, _, fg = dvr.render_backward(dv, f, kn, tf, prm, cams, T, k, torch.full_like(img, scale), want_features=True)
        e_max.append(abs(float(fg["gmax"]) / scale - rfg["gmax"]) / abs(rfg["gmax"]))
        e_tf.append(float(np.linalg.norm(dtf.cpu().numpy().astype(np.float64) / scale - rtf) / np.linalg.norm(rtf)))
    print(f"[sums] {shape} gmax {np.mean(e_max):.2e} ({max(e_max):.2e}) TF {np.mean(e_tf):.2e} ({max(e_tf):.2e})", flush=True)
    assert np.mean(e_max) <= 6e-7 and np.mean(e_tf) <= 1e-6
