"""FP32 network on the half-precision matrix cores (locc_detect in FP32 contexts): the sizes where its steps and tiles
end, the rows and weights out of the halves' range (computed as a chain of FP32 products), and the weights a training
step leaves.  Against the float64 oracle within 1e-5 per field, the FP32 tolerance of the other tests."""

import numpy as np
import pytest

from helpers import field_errors
from oracle import locc_oracle as O
from paper_2304_09439_amd import binding as B
from paper_2304_09439_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-5
NETS = {"small": I.SMALL_WIDTHS, "scale": I.SCALE_WIDTHS}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    B.load()
    return t


def _scene(n_pairs, n_points, seed=3):
    """Sphere pairs around contact and a few far apart: counts from 0 to the whole cloud."""
    rng = np.random.default_rng(seed)
    lib = I.sphere_library(rng, 12, n_points)
    s = rng.integers(0, 12, 2 * n_pairs).astype(np.int32)
    ta, qa, tb, qb = I.sphere_pair_poses(rng, lib.radius[s[0::2]], lib.radius[s[1::2]], 0.03)
    tb[::7] = ta[::7] + np.float32(0.5)
    pairs = np.arange(2 * n_pairs, dtype=np.int32).reshape(-1, 2)
    pairs[1::2] = pairs[1::2, ::-1]
    return I._pack_pair_scene(lib, ta, qa, tb, qb, s[0::2], s[1::2], pairs)


def _run(torch, scene, w, wd, K):
    ctx = B.context_for_scene(scene, K, wd, w)
    objs, pairs = B.scene_tensors(scene)
    out, counts = ctx.detect(objs, pairs)
    torch.cuda.synchronize()
    ctx.close()
    return out.cpu().numpy(), counts.cpu().numpy()


# 64-row steps and 32-row tiles (K, points per shape), 32-pair tiles, one or two of them per workgroup past 8,192 pairs
@pytest.mark.parametrize("net,K,points,pairs", [("small", 32, 33, 1), ("small", 256, 300, 33), ("scale", 96, 70, 31),
                                                ("scale", 160, 257, 65), ("scale", 64, 40, 8225)])
def test_split_forward_at_step_and_tile_edges(torch, net, K, points, pairs):
    w = NETS[net]
    wd = (w.h1, w.h2, w.hh)
    weights = I.flatten_weights(I.gaussian_weights(w, seed=2, bias_std=0.1))
    scene = _scene(pairs, points)
    out, counts = _run(torch, scene, weights, wd, K)
    rows = np.unique(np.concatenate([np.arange(min(pairs, 40)), np.arange(max(0, pairs - 40), pairs)]))
    ref = O.detect_scene(scene, weights, wd, K, rows=rows)
    np.testing.assert_array_equal(counts[rows], ref["counts"])
    assert max(field_errors(out[rows], ref["contacts"]).values()) < TOL
    alone, _ = _run(torch, scene.subset(rows), weights, wd, K)
    np.testing.assert_array_equal(alone, out[rows])   # whatever the batch


@pytest.mark.parametrize("net", ["small", "scale"])
def test_rows_out_of_the_halves_range(torch, net):
    """Unnormalised quaternions stretch the second object's normals past what the scales provide for: those pairs,
    and only those, take the FP32 chain."""
    w = NETS[net]
    wd = (w.h1, w.h2, w.hh)
    weights = I.flatten_weights(I.gaussian_weights(w, seed=2, bias_std=0.1))
    scene = _scene(70, 200)
    # 16 points of every cloud lie near its centre, so that some are in the crop however far the cloud is stretched
    rng = np.random.default_rng(1)
    pts = scene.lib.pts.reshape(12, 200, 6)
    pts[:, 60:76, :3] = rng.normal(0.0, 1e-5, (12, 16, 3))
    scene.pos[1::2] = scene.pos[0::2] + np.float32(0.01)
    plain, _ = _run(torch, scene, weights, wd, 96)
    odd = np.arange(70) % 5 == 2
    scene.quat[1::2][odd] *= np.float32(40.0)
    out, counts = _run(torch, scene, weights, wd, 96)
    np.testing.assert_array_equal(out[~odd], plain[~odd])
    ref = O.detect_scene(scene, weights, wd, 96)
    np.testing.assert_array_equal(counts, ref["counts"])
    assert (ref["counts"][odd] > 0).all() and np.abs(ref["z"][odd]).max() > 100   # rows past the halves' range
    assert max(field_errors(out[odd], ref["contacts"][odd]).values()) < TOL


@pytest.mark.parametrize("lr", [1e-3, 300.0])
def test_detect_after_training_uses_the_new_weights(torch, lr):
    """The halves follow the weights; weights grown past their scales (the large rate) take the FP32 chain."""
    w = I.SMALL_WIDTHS
    wd = (w.h1, w.h2, w.hh)
    scene = _scene(64, 200)
    ctx = B.context_for_scene(scene, 64, wd, I.flatten_weights(I.gaussian_weights(w, seed=4, bias_std=0.1)))
    objs, pairs = B.scene_tensors(scene)
    labels = torch.from_numpy((np.arange(64) % 2).astype(np.float32)).cuda()
    for _ in range(3):
        ctx.train_step(objs, pairs, labels, lr=lr)
    out, _ = ctx.detect(objs, pairs)
    trained = ctx.get_weights(0)
    torch.cuda.synchronize()
    ctx.close()
    ref = O.detect_scene(scene, trained, wd, 64)
    assert max(field_errors(out.cpu().numpy(), ref["contacts"]).values()) < TOL
