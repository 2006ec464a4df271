"""GPU parity of the render adjoint where several lanes share a ray (pixel pitches of about a voxel and
more, and images of few rays) against the oracle's reverse mode: dL/dTF, dL/dI and, with feature
gradients, dL/d(g, k, V, |g|_max).  The bar is the adjoint's own, 1e-4 normwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_19737_amd as dvr
import phantoms
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import f32, feats_np, oracle_params, sp32, to_dev

pytestmark = pytest.mark.gpu
TOL = 1e-4


def _norm(x, r):
    return float(np.linalg.norm(np.asarray(x, np.float64) - r) / np.linalg.norm(r))


# (dims, spacing, width, height, views, persp, K, et, step): 16 lanes by few rays; ragged images; 4 lanes
# by pitch (0.5-1.5 voxels a pixel) with more than 2^17 rays; 16 by pitch; thick slices; one segment a ray
CASES = [
    ((24, 20, 18), (1.0, 1.0, 1.0), 19, 13, 2, 0, 16, 0.0, 0.5),
    ((24, 20, 18), (1.0, 1.0, 1.0), 33, 21, 1, 1, 20, 0.9, 0.25),
    ((40, 36, 12), (0.6, 0.6, 4.0), 50, 47, 3, 1, 8, 0.9, 0.5),
    ((30, 28, 26), (1.0, 1.2, 0.9), 64, 70, 33, 0, 4, 0.0, 1.0),
    ((90, 80, 70), (1.0, 1.0, 1.0), 171, 130, 7, 0, 16, 0.99, 0.5),
    ((70, 64, 60), (1.0, 1.0, 1.0), 60, 40, 2, 0, 8, 0.0, 200.0),
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("layout", [abi.DVR_QUAD, abi.DVR_PLANAR, abi.DVR_INTERLEAVED])
def test_adjoint_lane_groups(case, layout):
    dims, h, W, H, views, persp, K, et, step = CASES[case]
    print(f"[lane groups] case {case} layout {layout}", flush=True)
    rng = np.random.default_rng(500 + case)
    # a smooth volume: intensities away from the TF knots except on thin shells
    z, y, x = np.meshgrid(*[np.linspace(0, 1, n) for n in dims[::-1]], indexing="ij")
    vol = (0.45 + 0.4 * np.sin(5 * x + 1) * np.cos(4 * y) * np.sin(3 * z + 0.5)).astype(np.float32)
    vol += 0.02 * rng.standard_normal(vol.shape).astype(np.float32)
    make = phantoms.persp_camera if persp else phantoms.ortho_camera
    cams = [make(dims, h, 360.0 * v / views + 20.0, 25.0, W, H) for v in range(views)]
    knots = np.linspace(0.0, 1.0, K).astype(np.float32)
    rgba = rng.uniform(0.1, 0.9, (K, 4)).astype(np.float32)
    rgba[:, 3] *= 0.3
    prm = phantoms.render_params(lambda_g=0.7, lambda_k=0.5, lambda_v=0.8, step_vox=step, et_alpha=et)
    dv = to_dev(vol)
    f = dvr.features(dv, h, [1.0], c=0.2, layout=layout).without_bricks()
    kn, tf = to_dev(knots), to_dev(rgba)
    sampled = dv if layout == abi.DVR_PLANAR else None
    img, T, k = dvr.render(sampled, f, kn, tf, prm, cams)
    dout = rng.standard_normal(tuple(img.shape)).astype(np.float32)
    dtf, dvol, fg = dvr.render_backward(sampled, f, kn, tf, prm, cams, T, k, to_dev(dout), want_features=True)
    ptf, pvol = dvr.render_backward(sampled, f, kn, tf, prm, cams, T, k, to_dev(dout))
    got = feats_np(f)
    # rays whose early termination falls on the other side in FP64 are left out of both
    ref = oracle.render(vol.astype(np.float64), got, got["gmax"], sp32(h), knots, rgba, oracle_params(prm), cams)
    flip = ref["k_last"] != k.cpu().numpy()
    assert flip.mean() < 1e-3
    if flip.any():
        dout[flip] = 0.0
        dtf, dvol, fg = dvr.render_backward(sampled, f, kn, tf, prm, cams, T, k, to_dev(dout), want_features=True)
        ptf, pvol = dvr.render_backward(sampled, f, kn, tf, prm, cams, T, k, to_dev(dout))
    rtf, rI, rfg, near = oracle.render_vjp(vol.astype(np.float64), got, got["gmax"], sp32(h), knots, rgba, oracle_params(prm),
                                           cams, dout, want_features=True, near_knot_eps=1e-6)
    keep = ~near  # the TF slope jumps at a knot: FP32 may take the neighbouring segment
    assert near.mean() < 0.05
    errs = dict(tf=_norm(dtf.cpu(), rtf), tf_plain=_norm(ptf.cpu(), rtf), I=_norm(dvol.cpu().numpy()[keep], rI[keep]),
                I_plain=_norm(pvol.cpu().numpy()[keep], rI[keep]), g=_norm(fg["g"].cpu(), rfg["g"]),
                kappa=_norm(fg["kappa"].cpu(), rfg["kappa"]), V=_norm(fg["V"].cpu(), rfg["V"]))
    errs["gmax"] = abs(float(fg["gmax"]) - rfg["gmax"]) / max(abs(rfg["gmax"]), np.abs(rfg["g"]).sum() * 1e-3)
    print("  " + " ".join(f"{n}={e:.1e}" for n, e in errs.items()), flush=True)
    assert max(errs.values()) <= TOL, errs


@pytest.mark.parametrize("layout", [abi.DVR_PLANAR, abi.DVR_INTERLEAVED, abi.DVR_SPLIT, abi.DVR_QUAD])
@pytest.mark.parametrize("dtype,et,bricks,persp,step", [
    (torch.float32, 0.99, False, True, 0.5), (torch.float32, 0.0, True, False, 0.37), (torch.float16, 0.9, True, True, 0.5)])
def test_forward_lane_groups_bit_identical(layout, dtype, et, bricks, persp, step):
    """The same views in one launch of 32 (one lane per ray), in launches of 4 (4 lanes) and one by one
    (16 lanes): image, ray state and sample counts agree bit for bit."""
    w = phantoms.c2(8, 8, views=[0])
    vol = to_dev(w.vol[40:100:2, 60:160:2, 30:150:2], dtype)
    h = (2.0, 2.0, 2.0)
    make = phantoms.persp_camera if persp else phantoms.ortho_camera
    cams = [make(tuple(vol.shape[::-1]), h, 11.25 * v, 15.0, 129, 101) for v in range(32)]
    kn, tf = to_dev(w.tf_knots), to_dev(w.tf_rgba)
    prm = dict(w.params, et_alpha=et, step_vox=step)
    print(f"[lane groups] forward layout {layout} {dtype} et {et}", flush=True)
    f = dvr.features(vol, h, [2.0], c=0.4, dtype=dtype, layout=layout)
    f = f if bricks else f.without_bricks()
    sampled = vol if layout in (abi.DVR_PLANAR, abi.DVR_SPLIT) else None

    def run(n):
        parts, total = [], torch.zeros(2, dtype=torch.int64, device="cuda")
        for i in range(0, 32, n):
            cnt = torch.zeros(2, dtype=torch.int64, device="cuda")
            parts.append(dvr.render(sampled, f, kn, tf, prm, cams[i:i + n], counters=cnt))
            total += cnt
        return [torch.cat([p[e] for p in parts]) for e in range(3)] + [total]

    one, four, sixteen = run(32), run(4), run(1)
    assert int(one[2].max()) > 16
    for other in (four, sixteen):
        for a, b in zip(one, other):
            assert torch.equal(a, b)
