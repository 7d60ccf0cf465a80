"""The FP32 network on the half-precision matrix cores where the magnitudes of a network, of a library or of a scene lie
far apart: margins and coordinates far above the other values, one large shape in a library, hidden units scaled
against the weights that read them, units that large biases keep at 0, and weights that training has made from zeros.
Against the float64 oracle within 1e-5 per field, the FP32 tolerance of the other tests."""

import numpy as np
import pytest

from helpers import field_errors
from oracle import locc_oracle as O
from paper_2304_09439_amd import binding as B
from paper_2304_09439_amd import inputs as I
from test_gpu_split import NETS, TOL, _scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    B.load()
    return t


def _layers(net, seed=2):
    return [a.copy() for a in I.gaussian_weights(NETS[net], seed=seed, bias_std=0.1)]


def _errors(torch, scene, net, layers, K, pad=O.PAD_M, rows=None):
    """Errors of detect's contacts, and of the contacts beside the pose gradients, over the pairs `rows`."""
    w = NETS[net]
    wd = (w.h1, w.h2, w.hh)
    flat = I.flatten_weights(layers)
    ctx = B.context_for_scene(scene, K, wd, flat, pad=pad)
    objs, pairs = B.scene_tensors(scene)
    out, counts = (t.cpu().numpy() for t in ctx.detect(objs, pairs))
    beside = ctx.pose_gradients(objs, pairs, want_contacts=True)[1].cpu().numpy()
    ctx.close()
    np.testing.assert_array_equal(beside, out)
    rows = np.arange(len(scene.pairs)) if rows is None else rows
    ref = O.detect_scene(scene, flat, wd, K, pad=pad, rows=rows)
    np.testing.assert_array_equal(counts[rows], ref["counts"])
    errs = field_errors(out[rows], ref["contacts"])
    print(net, pad, {k: f"{v:.1e}" for k, v in errs.items()}, flush=True)
    return max(errs.values())


@pytest.mark.parametrize("net", ["small", "scale"])
@pytest.mark.parametrize("pad", [1e3, 1e6, 1e9, 1e30])
def test_wide_margins(torch, net, pad):
    assert _errors(torch, _scene(64, 90), net, _layers(net), 96, pad) < TOL


@pytest.mark.parametrize("net", ["small", "scale"])
@pytest.mark.parametrize("distance", [3e2, 1e5, 1e9])
def test_far_objects_within_a_wide_margin(torch, net, distance):
    """The second object's rows have coordinates of the distance, the first's of its own size."""
    scene = _scene(64, 90)
    scene.pos[1::2] += (np.random.default_rng(5).normal(size=(64, 3)) * distance).astype(np.float32)
    assert _errors(torch, scene, net, _layers(net), 96, 100 * distance) < TOL


@pytest.mark.parametrize("net", ["small", "scale"])
@pytest.mark.parametrize("size", [1e3, 1e6, 1e12])
def test_one_large_shape_in_the_library(torch, net, size):
    """Shape 0 is larger than the others by far; half of the pairs have it, and one of its points is near them."""
    scene = _scene(64, 90)
    pts = scene.lib.pts.reshape(12, 90, 6)
    pts[0, 1:, :3] *= np.float32(size)
    rng = np.random.default_rng(6)
    pts[0, 5:40, :3] = rng.normal(0.0, 0.1, (35, 3))    # near points and far ones in one cloud
    scene.shape[:] = rng.integers(1, 12, 128)
    scene.shape[1:64:2] = 0
    scene.shape[64:96:2] = 0
    has = (scene.shape.reshape(-1, 2) == 0).any(axis=1)
    net_layers = _layers(net)
    assert _errors(torch, scene, net, net_layers, 96, rows=np.flatnonzero(~has)) < TOL
    assert _errors(torch, scene, net, net_layers, 96, rows=np.flatnonzero(has)) < TOL


UNITS = {"one": np.s_[3:4], "few": np.s_[0::9], "half": np.s_[0::2], "most": np.s_[4:]}


@pytest.mark.parametrize("net", ["small", "scale"])
@pytest.mark.parametrize("layer", [0, 1, 2, 3])
@pytest.mark.parametrize("k", [-30, -16, 20])
@pytest.mark.parametrize("units", list(UNITS))
def test_units_scaled_against_their_readers(torch, net, layer, k, units):
    """Hidden units times 2^k and the weights that read them times 2^-k: the same function."""
    L, u = _layers(net), UNITS[units]
    s = np.float32(2.0) ** k
    L[2 * layer][u] *= s
    L[2 * layer + 1][u] *= s
    reads = L[2 * layer + 2]
    if layer == 1:    # the features of both objects
        reads = reads.reshape(len(reads), 2, -1)
    reads[..., u] /= s
    assert _errors(torch, _scene(40, 90), net, L, 96) < TOL


@pytest.mark.parametrize("net", ["small", "scale"])
@pytest.mark.parametrize("layer", [0, 1, 2, 3])
@pytest.mark.parametrize("bias", [1e4, 1e7, 1e12])
def test_units_off_by_a_large_bias(torch, net, layer, bias):
    L = _layers(net)
    L[2 * layer + 1][1::5] = -bias
    assert _errors(torch, _scene(40, 90), net, L, 96) < TOL


@pytest.mark.parametrize("net", ["small", "scale"])
@pytest.mark.parametrize("layer", [1, 2, 3, 4])
def test_a_large_weight_of_an_idle_unit(torch, net, layer):
    """Every row of a matrix has one weight far above the others, of a unit that is always 0."""
    L = _layers(net)
    L[2 * layer - 2][7] = 0.0
    L[2 * layer - 1][7] = -1.0
    L[2 * layer][:, 7] = 1e6
    assert _errors(torch, _scene(40, 90), net, L, 96) < TOL


@pytest.mark.parametrize("net", ["small", "scale"])
def test_weights_trained_from_zero_and_shrunk(torch, net):
    """Rows that are zero at the upload and grow in training, and rows that shrink: the halves follow the weights."""
    w = NETS[net]
    wd = (w.h1, w.h2, w.hh)
    L = _layers(net, seed=4)
    L[2][3] = 0.0                # a row of the encoder's second layer,
    L[8][0], L[9][0] = 0.0, 0.0  # the logit's
    L[6][5] = 0.0                # and one of the head's
    L[4][9] *= np.float32(1e-4)  # weights of the size of one step, which may shrink to nothing
    scene = _scene(64, 200)
    ctx = B.context_for_scene(scene, 64, wd, I.flatten_weights(L))
    objs, pairs = B.scene_tensors(scene)
    labels = torch.from_numpy((np.arange(64) % 2).astype(np.float32)).cuda()
    for lr in (1e-4, 1e-5, 1e-6):
        for _ in range(3):
            ctx.train_step(objs, pairs, labels, lr=lr)
        out = ctx.detect(objs, pairs)[0].cpu().numpy()
        ref = O.detect_scene(scene, ctx.get_weights(0), wd, 64)
        errs = field_errors(out, ref["contacts"])
        print(net, lr, errs, flush=True)
        assert max(errs.values()) < TOL
    # a library uploaded after training does not bring the old weights' scales back
    ctx.upload_shapes(scene.lib.offsets, scene.lib.pts)
    np.testing.assert_array_equal(ctx.detect(objs, pairs)[0].cpu().numpy(), out)
    ctx.close()


@pytest.mark.parametrize("net", ["small", "scale"])
@pytest.mark.parametrize("k", [12, -12])
def test_a_library_in_another_unit(torch, net, k):
    """Shapes, poses and margin times 2^k and the weights of the coordinates times 2^-k: layer 1's products are the same
    bits, and so is what does not depend on the poses, whatever the unit: the halves', not the FP32 chains'."""
    w = NETS[net]
    wd = (w.h1, w.h2, w.hh)
    L, s = _layers(net), np.float32(2.0) ** k
    scene = _scene(64, 90)
    out = []
    for _ in range(2):
        ctx = B.context_for_scene(scene, 96, wd, I.flatten_weights(L), pad=0.01 if not out else 0.01 * float(s))
        objs, pairs = B.scene_tensors(scene)
        got, counts = (t.cpu().numpy() for t in ctx.detect(objs, pairs))
        out.append(np.concatenate([got[:, :1], got[:, 7:], counts], 1))
        ctx.close()
        scene.lib.pts[:, :3] *= s
        scene.pos *= s
        L[0][:, :3] /= s
    np.testing.assert_array_equal(out[0], out[1])
