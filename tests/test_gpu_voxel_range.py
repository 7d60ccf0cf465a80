"""The voxel variant's products of halves (the point MLP's layers 2 and 3, the predictor's hidden layers) where magnitudes
lie far apart: units scaled against the weights that read them, units that large biases keep at 0, a weight far above the
others of an idle unit, and one point far from a shape's others.  Against the float64 oracle, normwise within the 1e-4
of the other tests."""

import numpy as np
import pytest

from oracle import voxel_locc as V
from paper_2304_09439_amd import binding as B
from paper_2304_09439_amd import inputs as I
from test_gpu_voxel import TOL, _ctx, _normwise, _scene

pytestmark = pytest.mark.gpu

POINT = [0, 2]                       # arrays (weights, then biases) whose outputs products of halves read
PREDICTOR = [24, 26, 28, 30, 32]
UNITS = {"one": np.s_[3:4], "few": np.s_[0::9], "half": np.s_[0::2], "most": np.s_[4:]}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    B.load()
    return t


@pytest.fixture(scope="module")
def lib():
    full = I.scale_library(n_shapes=3)
    clouds = [full.pts[full.offsets[s]:full.offsets[s] + 200] for s in range(3)]
    return I.ShapeLibrary(np.concatenate(clouds), np.array([0, 200, 400, 600], np.int64), np.full(3, np.nan, np.float32))


@pytest.fixture(scope="module")
def plain(lib):
    """Embeddings and pairs' outputs of the weights that the tests change (most keep the function)."""
    return V.library_embeddings(lib.pts, lib.offsets, I.flatten_weights(_layers()))


def _layers():
    return [a.copy() for a in I.voxel_weights(seed=0, bias_std=0.1)]


def _embedding_error(lib, layers, emb=None, pts=None):
    flat = I.flatten_weights(layers)
    pts = lib.pts if pts is None else pts
    ref = V.library_embeddings(pts, lib.offsets, flat) if emb is None else emb
    ctx = B.VoxelContext()
    ctx.upload_weights(flat)
    ctx.upload_shapes(lib.offsets, pts)
    got = ctx.embeddings().cpu().numpy()
    ctx.close()
    errs = [_normwise(got[s], ref[s]) for s in range(lib.n_shapes)]
    print(["%.1e" % e for e in errs], flush=True)
    return max(errs)


def _pair_error(torch, lib, layers, emb):
    flat = I.flatten_weights(layers)
    pos, quat, shape, pairs = _scene(lib, n_pairs=80)
    ref = V.detect(lib.pts, lib.offsets, pos, quat, shape, pairs, flat, emb=emb)
    ctx = _ctx(lib, flat)
    objs = torch.from_numpy(B.pack_objects(pos, quat, shape)).cuda()
    out = ctx.detect(objs, torch.from_numpy(pairs).cuda())[0].cpu().numpy()
    ctx.close()
    ok = ~np.isnan(ref["logit"])
    err = _normwise(out[ok, 0], ref["logit"][ok])
    print("%.1e" % err, flush=True)
    return err


def _error(torch, lib, layers, emb, array):
    return _embedding_error(lib, layers, emb) if array < 6 else _pair_error(torch, lib, layers, emb)


@pytest.mark.parametrize("array", POINT + PREDICTOR)
@pytest.mark.parametrize("k", [-45, -24, 24])
@pytest.mark.parametrize("units", list(UNITS))
def test_units_scaled_against_their_readers(torch, lib, plain, array, k, units):
    L, u, s = _layers(), UNITS[units], np.float32(2.0) ** k
    L[array][u] *= s
    L[array + 1][u] *= s
    L[array + 2][:, u] /= s
    assert _error(torch, lib, L, plain, array) < TOL


@pytest.mark.parametrize("array", POINT + PREDICTOR)
@pytest.mark.parametrize("bias", [1e7, 1e12])
def test_units_off_by_a_large_bias(torch, lib, plain, array, bias):
    L = _layers()
    L[array + 1][1::5] = -bias
    assert _error(torch, lib, L, None if array < 6 else plain, array) < TOL


@pytest.mark.parametrize("array", POINT + PREDICTOR)
def test_a_large_weight_of_an_idle_unit(torch, lib, plain, array):
    L = _layers()
    L[array][7] = 0.0
    L[array + 1][7] = -1.0
    L[array + 2][:, 7] = 1e8
    assert _error(torch, lib, L, None if array < 6 else plain, array) < TOL


@pytest.mark.parametrize("size", [1e4, 1e8])
def test_one_far_point_in_a_shape(torch, lib, size):
    """The far point has a cell of its own, and every channel of the map reads the near ones' cell alone (the far
    point's features are switched off by a bias far below them)."""
    L = _layers()
    pts = lib.pts.copy()
    pts[0::200, :3] = size
    # layer 1 falls along (1, 1, 1), so that the far point's outputs are 0 everywhere
    L[0][:] = np.abs(L[0]) * -1.0
    L[1][:] = np.abs(L[1]) + 0.5
    assert _embedding_error(lib, L, pts=pts) < TOL
