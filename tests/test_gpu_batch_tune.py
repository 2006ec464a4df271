"""The ray tiles of a batched launch and their autotuner.  The tile shapes the rays of a wave only where a view
takes one lane per ray (more than 1.2 M rays in the batch, at most 0.6 voxels a pixel): there every shape gives
the standalone calls' images and ray state bit for bit, on odd image sizes.  Where no view does, the
autotuner has nothing to time, leaves the outputs alone and its cache entry has no say in other batches."""
import json

import numpy as np
import pytest
import torch

import paper_2605_19737_amd as dvr
import phantoms
from paper_2605_19737_amd import _abi as abi
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu
SP = (1.0, 1.1, 1.4)


def _scene(sizes, layout, dtype):
    rng = np.random.default_rng(11)
    w = phantoms.c4_volume(0, 64, 64)
    shapes = [(40, 44, 50), (22, 60, 36)]
    vols = [to_dev(rng.random(s, dtype=np.float32), dtype) for s in shapes]
    feats = [dvr.alloc_features(s, SP, dtype, layout) for s in shapes]
    views = []
    for i, s in enumerate(shapes):
        for j, (W, H) in enumerate(sizes):
            cam = phantoms.ortho_camera(s[::-1], SP, 40.0 * i + 70.0 * j, 25.0, W, H)
            views.append((i, cam, torch.full((H, W, 4), -1.0, device="cuda"), torch.empty((H, W), device="cuda"),
                          torch.empty((H, W), dtype=torch.int32, device="cuda")))
    return w, vols, feats, views, to_dev(w.tf_knots), to_dev(w.tf_rgba)


@pytest.mark.parametrize("layout,dtype", [(abi.DVR_SPLIT, torch.float32), (abi.DVR_INTERLEAVED, torch.float32),
                                          (abi.DVR_QUAD, torch.float16)])
def test_ray_tiles_equal_standalone(layout, dtype, tmp_path):
    w, vols, feats, views, kn, tf = _scene([(1003, 701), (331, 417), (18, 33)], layout, dtype)
    cache = str(tmp_path / "tune.json")
    best = dvr.Batch.autotune(vols, [SP] * 2, feats, views, [1.0], kn, tf, w.params, c=w.c, cache_path=cache)
    assert not any(k.endswith("|shared") for k in json.load(open(cache)))  # a view takes one lane per ray
    tunes = [dict(wg_per_cu=4, xy_tile=0, xy_zrun=32, z_chunk=8, ray_tile=r) for r in range(3)]
    assert best in tunes
    refs = []
    for i, cam, _, _, _ in views:
        f = dvr.features(vols[i], SP, [1.0], c=w.c, dtype=dtype, layout=layout)
        sv = vols[i] if layout == abi.DVR_SPLIT else None
        refs.append(dvr.render(sv, f.without_bricks(), kn, tf, w.params, [cam]))
    for tune in tunes:
        print(f"[batch tune] layout {layout} ray_tile {tune['ray_tile']}", flush=True)
        b = dvr.Batch(vols, [SP] * 2, feats, views, [1.0], kn, tf, w.params, c=w.c, tune=tune)
        for v in views:
            v[2].fill_(-1.0)
        b.launch()
        b.check()
        for (_, _, img, T, k), (rimg, rT, rk) in zip(views, refs):
            assert torch.equal(img, rimg[0]) and torch.equal(T, rT[0]) and torch.equal(k, rk[0])
        b.close()


def test_autotune_without_a_one_lane_view(tmp_path):
    w, vols, feats, views, kn, tf = _scene([(96, 80)], abi.DVR_SPLIT, torch.float32)
    cache = str(tmp_path / "tune.json")
    args = (vols, [SP] * 2, feats, views, [1.0], kn, tf, w.params)
    default = dict(wg_per_cu=4, xy_tile=0, xy_zrun=32, z_chunk=8, ray_tile=0)
    assert dvr.Batch.autotune(*args, c=w.c, cache_path=cache) == default
    torch.cuda.synchronize()
    assert all(bool((v[2] == -1.0).all()) for v in views)
    entries = json.load(open(cache))
    (key,) = entries
    assert key.endswith("|shared")
    # an entry of a batch of this class whose views take one lane, and the other way round
    with open(cache, "w") as f:
        f.write("{\n  \"%s\": [4, 0, 32, 8, 2]\n}\n" % key[: -len("|shared")])
    assert dvr.Batch.autotune(*args, c=w.c, cache_path=cache) == default
    assert sorted(json.load(open(cache))) == sorted([key, key[: -len("|shared")]])
    with pytest.raises(dvr.DVRError):
        dvr.Batch.autotune(vols, [SP] * 2, feats, views, [1.0], kn, tf, w.params, c=-1.0)
