"""Views of which a small volume covers a few pixels, at pitches that give a ray several lanes: rays and
workgroups that meet nothing must add nothing and cost next to nothing.  The same rays are taken once from a
large image and once from its middle alone: the images agree bit for bit, the gradients within the adjoint's
bar of 1e-4 (normwise), and the large image does not take several times as long."""
import numpy as np
import pytest
import torch

import paper_2605_19737_amd as dvr
import phantoms
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu
W, H, X0, Y0, SIDE = 1000, 700, 440, 290, 128  # the image, and the window of SIDE^2 around its middle
D0 = np.array((0.25, 0.125, 1.0), np.float32) / np.float32(np.sqrt(1.078125))


def _cams(pitch, views):
    """Orthographic views at FP32-exact origins, with and without the pixels around the window."""
    out = []
    for v in range(views):
        du, dv = np.array((pitch, 0, 0), np.float32), np.array((0, pitch, 0), np.float32)
        o = np.array((-500.0 * pitch + 4.0 * v, -350.0 * pitch, -32.0), np.float32)
        d0 = D0 * np.array((1, -1 if v & 1 else 1, 1), np.float32)
        out.append((phantoms.Camera(0, W, H, o, d0, du, dv), phantoms.Camera(0, SIDE, SIDE, o + X0 * du + Y0 * dv, d0, du, dv)))
    return [c[0] for c in out], [c[1] for c in out]


def _scene(shape, layout, K):
    rng = np.random.default_rng(K)
    z, y, x = np.meshgrid(*[np.linspace(0, 1, n) for n in shape], indexing="ij")
    vol = to_dev((0.45 + 0.4 * np.sin(5 * x + 1) * np.cos(4 * y) * np.sin(3 * z + 0.5)).astype(np.float32))
    rgba = rng.uniform(0.1, 0.9, (K, 4)).astype(np.float32)
    rgba[:, 3] *= 0.3
    f = dvr.features(vol, (1.0, 1.0, 1.0), [1.0], c=0.2, layout=layout).without_bricks()
    prm = phantoms.render_params(lambda_g=0.7, lambda_k=0.5, lambda_v=0.8, step_vox=0.5, et_alpha=0.99)
    return (vol if layout in (abi.DVR_PLANAR, abi.DVR_SPLIT) else None), f, to_dev(np.linspace(0, 1, K).astype(np.float32)), \
        to_dev(rgba), prm


def _us(f):
    f()
    best = float("inf")
    for _ in range(5):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(10):
            f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 100.0)
    return best


def _norm(a, b):
    return float((a - b).norm() / b.norm())


@pytest.mark.parametrize("layout,K", [(abi.DVR_QUAD, 8), (abi.DVR_PLANAR, 20), (abi.DVR_SPLIT, 16)])
@pytest.mark.parametrize("pitch", [1.0, 4.0])
def test_adjoint_of_sparse_views(layout, K, pitch):
    sv, f, kn, tf, prm = _scene((30, 36, 40), layout, K)
    large, middle = _cams(pitch, 3)
    print(f"[sparse] adjoint layout {layout} K {K} pitch {pitch}", flush=True)
    img, T, k = dvr.render(sv, f, kn, tf, prm, large)
    crop, Tc, kc = dvr.render(sv, f, kn, tf, prm, middle)
    win = (slice(None), slice(Y0, Y0 + SIDE), slice(X0, X0 + SIDE))
    assert torch.equal(img[win], crop) and torch.equal(T[win], Tc) and torch.equal(k[win], kc)
    assert int((k >= 0).sum()) == int((kc >= 0).sum()) > 50
    g = torch.randn_like(img)
    gc = g[win].contiguous()
    tf1, vol1, fg1 = dvr.render_backward(sv, f, kn, tf, prm, large, T, k, g, want_features=True)
    tf2, vol2, fg2 = dvr.render_backward(sv, f, kn, tf, prm, middle, Tc, kc, gc, want_features=True)
    ptf, pvol = dvr.render_backward(sv, f, kn, tf, prm, large, T, k, g)
    errs = [_norm(tf1, tf2), _norm(vol1, vol2), _norm(fg1["packed"], fg2["packed"]), _norm(ptf, tf2), _norm(pvol, vol2)]
    print("  " + " ".join(f"{e:.1e}" for e in errs), flush=True)
    assert max(errs) <= 1e-4


def test_adjoint_of_sparse_views_is_not_slow():
    sv, f, kn, tf, prm = _scene((6, 56, 60), abi.DVR_SPLIT, 8)
    large, middle = _cams(4.0, 3)
    t = []
    for cams in (large, middle):
        img, T, k = dvr.render(sv, f, kn, tf, prm, cams)
        g = torch.randn_like(img)
        t.append(_us(lambda: dvr.render_backward(sv, f, kn, tf, prm, cams, T, k, g)))
    print(f"[sparse] adjoint, large image {t[0]:.1f} us, its middle {t[1]:.1f} us", flush=True)
    assert t[0] <= 4.0 * t[1]


def test_render_of_sparse_views_is_not_slow():
    """A ray that misses costs a set-up for each of its lanes, so a volume that is small in its image keeps
    fewer of them."""
    sv, f, kn, tf, prm = _scene((6, 56, 60), abi.DVR_SPLIT, 20)
    large, middle = _cams(4.0, 1)
    t = []
    for cams in (large, middle):
        img = dvr.render(sv, f, kn, tf, prm, cams)[0]
        t.append(_us(lambda: dvr.render(sv, f, kn, tf, prm, cams, want_state=False, out=img)))
    print(f"[sparse] render, large image {t[0]:.1f} us, its middle {t[1]:.1f} us", flush=True)
    assert t[0] <= 4.0 * t[1]
