"""Images of 2^30 pixels at a coarse pitch, where the lanes that a smaller image gives each ray would need more
threads than a grid holds: the raymarch against the FP64 oracle on the pixels around the volume, which lies
near the last row and column, with every pixel elsewhere exactly zero."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_19737_amd as dvr
import phantoms
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import compare_images, f32, feats_np, oracle_params, sp32, to_dev

pytestmark = pytest.mark.gpu
SIDE, EDGE = 32768, 32680  # the box covers about 14 pixels on from EDGE + 20
SHAPE, SP = (9, 12, 14), (1.0, 1.0, 1.0)


def _camera():
    e = np.eye(3, dtype=np.float32)  # a voxel a pixel
    o = np.array((-(EDGE + 20.0), -(EDGE + 20.0), -5.0), np.float32)
    return phantoms.Camera(0, SIDE, SIDE, o, e[2], e[0], e[1])


def _check(vol, feats, w, cam, img, T, k, label):
    assert not bool(img[:EDGE].any()) and not bool(img[EDGE:, :EDGE].any())
    j, i = np.meshgrid(np.arange(EDGE, SIDE), np.arange(EDGE, SIDE), indexing="ij")
    pix = np.stack([np.zeros(i.size), i.ravel(), j.ravel()], 1).astype(np.int32)
    f = feats_np(feats)
    ref = oracle.render(vol.cpu().numpy().astype(np.float64), f, f["gmax"], sp32(SP), w.tf_knots, w.tf_rgba,
                        oracle_params(w.params), [cam], pix=pix)
    assert (ref["k_last"] >= 0).sum() > 100
    at = pix.copy()
    at[:, 1:] -= EDGE
    compare_images(img[None, EDGE:, EDGE:], T[None, EDGE:, EDGE:], k[None, EDGE:, EDGE:], ref,
                   f32(w.params["et_alpha"]), label, pix=at)


def _scene():
    w = phantoms.c4_volume(0, 64, 64)
    vol = to_dev(np.random.default_rng(3).random(SHAPE, dtype=np.float32))
    return w, vol, to_dev(w.tf_knots), to_dev(w.tf_rgba)


def test_render_of_2_30_pixels():
    w, vol, kn, tf = _scene()
    cam = _camera()
    f = dvr.features(vol, SP, [1.0], c=w.c, layout=abi.DVR_QUAD).without_bricks()
    print(f"[large] render {SIDE}^2", flush=True)
    img, T, k = dvr.render(None, f, kn, tf, w.params, [cam])
    _check(vol, f, w, cam, img[0], T[0], k[0], "2^30 pixels")


def test_batch_view_of_2_30_pixels():
    w, vol, kn, tf = _scene()
    cam = _camera()
    f = dvr.alloc_features(SHAPE, SP, layout=abi.DVR_QUAD, bricks=False)
    img = torch.full((SIDE, SIDE, 4), -1.0, dtype=torch.float32, device="cuda")
    T = torch.empty((SIDE, SIDE), dtype=torch.float32, device="cuda")
    k = torch.empty((SIDE, SIDE), dtype=torch.int32, device="cuda")
    print(f"[large] batched view {SIDE}^2", flush=True)
    b = dvr.Batch([vol], [SP], [f], [(0, cam, img, T, k)], [1.0], kn, tf, w.params, c=w.c)
    b.launch()
    b.check()
    _check(vol, f, w, cam, img, T, k, "2^30 pixels, batched")
    b.close()
