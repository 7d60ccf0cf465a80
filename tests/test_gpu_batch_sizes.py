"""BF16 and FP8 detect at the batch sizes where the launches change: one pair per workgroup, shares, the pair set-up inside
or ahead of the crop, the encoder and the
head as kernels of their own (scale widths), two row tiles per head workgroup.  Every pair is computed on its own with
the same operations whatever the batch, so a batch must equal its parts, computed in small batches, bit for bit."""

import numpy as np
import pytest

from oracle import locc_oracle as O
from paper_2304_09439_amd import binding as B
from paper_2304_09439_amd import inputs as I
from test_gpu_split import NETS, _scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    B.load()
    return t


@pytest.mark.parametrize("precision", ["bf16", "fp8_encoder"])
@pytest.mark.parametrize("net,K,sizes", [("small", 32, (1, 257, 1025)),
                                         ("scale", 32, (1, 1023, 1025, 2048, 2049, 4097)),
                                         ("scale", 96, (31, 1024, 1055, 4095, 12289))])
def test_batches_equal_their_parts(torch, precision, net, K, sizes):
    w = NETS[net]
    wd = (w.h1, w.h2, w.hh)
    weights = I.flatten_weights(I.gaussian_weights(w, seed=4, bias_std=0.1))
    scene = _scene(max(sizes), K + 9)
    scene.pairs[5] = (3, 3)  # an invalid pair
    ctx = B.context_for_scene(scene, K, wd, weights, precision=precision)
    objs, pairs = B.scene_tensors(scene)
    if precision != "bf16":
        ctx.calibrate(objs, pairs[:256])
    whole = [t.cpu().numpy() for t in ctx.debug_forward(objs, pairs)]
    for n in sizes[:-1]:
        part = [t.cpu().numpy() for t in ctx.debug_forward(objs, pairs[:n].contiguous())]
        for a, b in zip(part, whole):
            np.testing.assert_array_equal(a, b[:n])
    tail = [t.cpu().numpy() for t in ctx.debug_forward(objs, pairs[-40:].contiguous())]
    for a, b in zip(tail, whole):
        np.testing.assert_array_equal(a, b[-40:])
    # an actual count in device memory below the capacity: the rest stays untouched
    out = torch.full((max(sizes), 8), 7.0, device=objs.device)
    n_dev = torch.tensor([max(sizes) - 33], dtype=torch.int32, device=objs.device)
    ctx.detect_device_count(objs, pairs, n_dev, out)
    got = out.cpu().numpy()
    np.testing.assert_array_equal(got[:-33], whole[0][:-33])
    assert (got[-33:] == 7.0).all()
    ctx.close()
    rows = np.r_[0:5, 6:30]
    ref = O.detect_scene(scene, weights, wd, K, rows=rows)
    np.testing.assert_array_equal(whole[1][rows], ref["counts"])
    # bf16 rounds inputs, weights and activations of five layers to 2^-9 each, e4m3 one layer to 2^-4
    err = np.abs(whole[2][rows] - ref["z"]).max() / np.abs(ref["z"]).max()
    assert err < (0.02 if precision == "bf16" else 0.1)


@pytest.mark.parametrize("net,K,sizes", [("small", 32, (511, 513, 2048, 2049, 12288, 12289)),
                                         ("scale", 32, (255, 257, 1024, 1025, 2049))])
def test_fp32_batches_equal_their_parts(torch, net, K, sizes):
    """One claim per workgroup or the queue's; argmax chains of one object or of four per workgroup."""
    w = NETS[net]
    wd = (w.h1, w.h2, w.hh)
    weights = I.flatten_weights(I.gaussian_weights(w, seed=4, bias_std=0.1))
    scene = _scene(max(sizes), K + 9)
    ctx = B.context_for_scene(scene, K, wd, weights)
    objs, pairs = B.scene_tensors(scene)
    whole = [t.cpu().numpy() for t in ctx.detect(objs, pairs)]
    grad, out, arg = ctx.pose_gradients(objs, pairs, want_contacts=True, want_argmax=True)
    grads = [t.cpu().numpy() for t in (grad, out, arg)]
    for n in sizes[:-1]:
        part = pairs[:n].contiguous()
        for a, b in zip(ctx.detect(objs, part), whole):
            np.testing.assert_array_equal(a.cpu().numpy(), b[:n])
        for a, b in zip(ctx.pose_gradients(objs, part, want_contacts=True, want_argmax=True), grads):
            np.testing.assert_array_equal(a.cpu().numpy().reshape(-1), b.reshape(len(pairs), -1)[:n].reshape(-1))
    out = torch.full((max(sizes), 8), 7.0, device=objs.device)
    n_dev = torch.tensor([max(sizes) - 33], dtype=torch.int32, device=objs.device)
    ctx.detect_device_count(objs, pairs, n_dev, out)
    got = out.cpu().numpy()
    np.testing.assert_array_equal(got[:-33], whole[0][:-33])
    assert (got[-33:] == 7.0).all()
    ctx.close()


@pytest.mark.parametrize("precision", ["bf16", "fp8_encoder"])
def test_small_batches_equal_their_parts(torch, precision):
    """The head as a kernel of its own from one pair in two compute units on, with two tiles a workgroup past one tile a
    compute unit; the FP8 encoder's third workgroup, and the batches that do without it."""
    test_batches_equal_their_parts(torch, precision, "scale", 64,
                                   (127, 128, 129, 256, 257, 513, 769, 3072, 3073, 4608, 4609, 8192, 8193))
