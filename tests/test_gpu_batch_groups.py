"""Batched launch of small volumes, whose feature passes share launches: volumes of odd and uneven sizes (2 voxels
to a size class of their own), spacings that give several stencil radii in the plane and along z, and, among
them, volumes that cannot share (in-plane radii that differ, a radius above 10, more than 2^20 voxels).  The
values are the standalone calls', bit for bit, in every dtype and layout and on every replay; and the launches
are shared: 256 volumes of 24^3 take no more than a few times what one volume of their voxels takes."""
import numpy as np
import pytest
import torch

import paper_2605_19737_amd as dvr
import phantoms
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu
A, B, C = (0.7, 0.7, 1.9), (1.0, 1.0, 1.0), (0.5, 0.5, 0.4)
SET = [((19, 33, 41), A), ((2, 2, 2), A), ((24, 9, 17), B), ((5, 48, 70), A), ((12, 12, 70), C), ((31, 21, 11), B),
       ((16, 16, 130), A), ((40, 40, 40), C), ((300, 2, 3), B), ((24, 30, 28), (0.7, 0.9, 1.0)), ((9, 20, 22), (0.28, 0.28, 0.6)),
       ((70, 120, 130), B), ((64, 64, 64), A)]


def _views(shapes, spacings, side):
    cams = [phantoms.ortho_camera(s[::-1], sp, 30.0 * i, 20.0, side, side + 5) for i, (s, sp) in enumerate(zip(shapes, spacings))]
    return [(i, c, torch.empty((side + 5, side, 4), device="cuda"), torch.empty((side + 5, side), device="cuda"),
             torch.empty((side + 5, side), dtype=torch.int32, device="cuda")) for i, c in enumerate(cams)]


@pytest.mark.parametrize("layout", [abi.DVR_PLANAR, abi.DVR_INTERLEAVED, abi.DVR_SPLIT, abi.DVR_QUAD])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("sigmas", [[1.0], [0.6, 1.3]])
def test_shared_launches_equal_standalone(layout, dtype, sigmas):
    print(f"[batch groups] layout {layout} {dtype} {sigmas}", flush=True)
    rng = np.random.default_rng(7)
    w = phantoms.c4_volume(0, 64, 64)
    shapes, sps = [s for s, _ in SET], [h for _, h in SET]
    vols = [to_dev(rng.random(s, dtype=np.float32), dtype) for s in shapes]
    feats = [dvr.alloc_features(s, h, dtype, layout) for s, h in SET]
    kn, tf = to_dev(w.tf_knots), to_dev(w.tf_rgba)
    views = _views(shapes, sps, 21)
    b = dvr.Batch(vols, sps, feats, views, sigmas, kn, tf, w.params, c=w.c)
    for rep in range(3):
        for f in feats:
            f.grad.fill_(7.0)
            f.gmax.fill_(7.0)
        for v in views:
            v[2].fill_(-1.0)
        b.launch()
        b.check()
        torch.cuda.synchronize()
        for (i, cam, img, T, k), vol, h, f in zip(views, vols, sps, feats):
            r = dvr.features(vol, h, sigmas, c=w.c, dtype=dtype, layout=layout)
            for name in ("grad", "kappa", "ves", "iquad", "gmax"):
                x, y = getattr(f, name), getattr(r, name)
                assert (x is None and y is None) or torch.equal(x, y), (rep, i, name)
            sv = vol if layout in (abi.DVR_PLANAR, abi.DVR_SPLIT) else None
            rimg, rT, rk = dvr.render(sv, r, kn, tf, w.params, [cam])
            assert torch.equal(img, rimg[0]) and torch.equal(T, rT[0]) and torch.equal(k, rk[0]), (rep, i)
    b.close()


def test_more_volumes_than_one_group_holds():
    """21 volumes of 101^3 (1.03 M voxels each): four fill a group of 2^22 voxels, so there are six, on four branches."""
    shape, h = (101, 101, 101), (1.0, 1.0, 1.0)
    w = phantoms.c4_volume(0, 64, 64)
    g = torch.Generator(device="cuda").manual_seed(3)
    vols = [torch.rand(shape, generator=g, device="cuda") for _ in range(21)]
    feats = [dvr.alloc_features(shape, h, layout=abi.DVR_SPLIT, bricks=False) for _ in vols]
    kn, tf = to_dev(w.tf_knots), to_dev(w.tf_rgba)
    b = dvr.Batch(vols, [h] * 21, feats, [], [1.0, 1.5], kn, tf, w.params, c=w.c)
    for _ in range(2):
        b.launch()
        b.check()
        for v, f in zip(vols, feats):
            r = dvr.features(v, h, [1.0, 1.5], c=w.c, layout=abi.DVR_SPLIT)
            assert torch.equal(f.grad, r.grad) and torch.equal(f.ves, r.ves) and torch.equal(f.gmax, r.gmax)
    b.close()


def test_a_volume_of_more_slices_than_a_grid_has():
    """Two volumes of 70000 slices, one beside small ones and one above 2^20 voxels: runs of their
    slices equal the features of a copy of those 80 slices alone, away from the copy's ends."""
    w = phantoms.c4_volume(0, 64, 64)
    g = torch.Generator(device="cuda").manual_seed(5)
    h, shapes = (1.0, 1.0, 1.0), [(70000, 2, 3), (70000, 4, 4), (20, 20, 20)]
    vols = [torch.rand(s, generator=g, device="cuda") for s in shapes]
    feats = [dvr.alloc_features(s, h, layout=abi.DVR_SPLIT, bricks=False) for s in shapes]
    kn, tf = to_dev(w.tf_knots), to_dev(w.tf_rgba)
    print("[batch groups] 70000 slices", flush=True)
    b = dvr.Batch(vols, [h] * 3, feats, [], [1.0], kn, tf, w.params, c=w.c)
    b.launch()
    b.check()
    R = 4  # stencil radius at sigma 1
    for v, f in zip(vols[:2], feats[:2]):
        n = v.shape[0]
        for z0 in (0, 33333, 65500, n - 80):
            part = v[z0:z0 + 80].clone()
            r = dvr.features(part, h, [1.0], c=w.c, layout=abi.DVR_SPLIT)
            lo, hi = (0 if z0 == 0 else R), (80 if z0 + 80 == n else 80 - R)
            assert torch.equal(f.grad[z0 + lo:z0 + hi], r.grad[lo:hi]) and torch.equal(f.ves[z0 + lo:z0 + hi], r.ves[lo:hi])
    b.close()


def _us(f):
    f()
    best = float("inf")
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(5):
            f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 200.0)
    return best


def test_many_small_volumes_are_not_slow():
    w = phantoms.c4_volume(0, 64, 64)
    kn, tf = to_dev(w.tf_knots), to_dev(w.tf_rgba)
    t = []
    for n, shape in ((256, (24, 24, 24)), (1, (152, 152, 153))):
        h = (1.0, 1.0, 1.0)
        vols = [torch.rand(shape, device="cuda") for _ in range(n)]
        feats = [dvr.alloc_features(shape, h, layout=abi.DVR_SPLIT, bricks=False) for _ in vols]
        b = dvr.Batch(vols, [h] * n, feats, [], [1.0], kn, tf, w.params, c=w.c)
        t.append(_us(b.launch))
        b.check()
        b.close()
    print(f"[batch groups] 256 volumes of 24^3 {t[0]:.0f} us, one of their voxels {t[1]:.0f} us", flush=True)
    assert t[0] <= 5.0 * t[1]
