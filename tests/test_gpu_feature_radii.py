"""GPU parity of the fixed-radius feature kernels and their adjoint at the largest stencil radii
(11..15), and of the storage types and layouts that share one kernel, against the FP64 oracle with
the feature pass's own bars (1e-5 of each output's range; adjoint 1e-4 normwise)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_19737_amd as dvr
import phantoms
from oracle import feature_adjoint as fa
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import compare_features, f32, feats_np, sp32, to_dev

pytestmark = pytest.mark.gpu


def _crop():
    return phantoms.c2(8, 8, views=[0]).vol[60:91, 70:107, 40:125]


@pytest.mark.parametrize("radius", [11, 12, 13, 14, 15])
@pytest.mark.parametrize("layout", [abi.DVR_PLANAR, abi.DVR_INTERLEAVED])
def test_features_large_radius(radius, layout):
    vol, sg = _crop(), (radius - 1) / 3.0
    print(f"[features] radius {radius} layout {layout}", flush=True)
    f = dvr.features(to_dev(vol), (1.0, 1.0, 1.0), [sg], c=0.4, layout=layout)
    ref = oracle.features(vol.astype(np.float64), (1.0, 1.0, 1.0), [f32(sg)], c=f32(0.4), want_lam=True)
    compare_features(feats_np(f), ref, f"radius {radius}")


@pytest.mark.parametrize("vol_dt,out_dt,layout", [
    (torch.float32, torch.float32, abi.DVR_INTERLEAVED), (torch.float32, torch.float16, abi.DVR_PLANAR),
    (torch.float32, torch.float16, abi.DVR_SPLIT), (torch.float16, torch.float32, abi.DVR_PLANAR),
    (torch.float16, torch.float32, abi.DVR_SPLIT), (torch.float16, torch.float16, abi.DVR_PLANAR)])
def test_features_shared_kernel_storage(vol_dt, out_dt, layout):
    """Two scales (the second reads the first's stored V), ragged tiles; FP16 storage within 2^-11 of
    the range on top of the compute bar."""
    print(f"[features] {vol_dt} -> {out_dt} layout {layout}", flush=True)
    dv = to_dev(_crop()).to(vol_dt)
    sg = [1.0, 2.0]
    f = dvr.features(dv, (0.9, 0.9, 1.3), sg, c=0.4, dtype=out_dt, layout=layout)
    ref = oracle.features(dv.float().cpu().numpy().astype(np.float64), sp32((0.9, 0.9, 1.3)), sg, c=f32(0.4), want_lam=True)
    compare_features(feats_np(f), ref, "shared", tol=1e-5 + (2.0 ** -11 if out_dt == torch.float16 else 0.0))


@pytest.mark.parametrize("radius", [11, 15])
def test_feature_adjoint_large_radius(radius):
    rng = np.random.default_rng(radius)
    vol = _crop()[:, :21, :70]
    sg = (radius - 1) / 3.0
    up = dict(g=rng.standard_normal((3,) + vol.shape), kappa=rng.standard_normal(vol.shape), V=rng.standard_normal(vol.shape))
    print(f"[feature adjoint] radius {radius}", flush=True)
    got = dvr.features_backward(to_dev(vol), (1.0, 1.0, 1.0), [sg],
                                dict({k: to_dev(v) for k, v in up.items()}, gmax=to_dev(np.array([0.7]))), c=0.4)
    ref = fa.vjp(vol.astype(np.float64), (1.0, 1.0, 1.0), [f32(sg)], 0.5, 0.5, f32(0.4),
                 *(up[k].astype(np.float32).astype(np.float64) for k in ("g", "kappa", "V")), f32(0.7))
    err = np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"  err {err:.2e}", flush=True)
    assert err <= 1e-4
