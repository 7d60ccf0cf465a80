"""The crop's scan by spatial clusters: index sets and counts of shapes whose last cluster is full, nearly empty or just
begun, of shapes of equal and of coplanar points, in batches on both sides of the size rule, equal the oracle's exactly;
without counts, where a scan may end early, the contacts are those of the run with counts, bit for bit."""

import numpy as np
import pytest

from oracle import locc_oracle as O
from paper_2304_09439_amd import binding as B
from paper_2304_09439_amd import inputs as I

pytestmark = pytest.mark.gpu
WD = (I.SMALL_WIDTHS.h1, I.SMALL_WIDTHS.h2, I.SMALL_WIDTHS.hh)


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a GPU"
    B.load()
    return t


def _scene(sizes, n_pairs, seed):
    rng = np.random.default_rng(seed)
    half = rng.uniform(0.05, 0.3, (len(sizes) + 2, 3))
    pts = [np.concatenate([rng.uniform(-h, h, (m, 3)), rng.normal(size=(m, 3))], 1) for h, m in zip(half, sizes)]
    pts.append(np.tile(np.array([[0.05, -0.02, 0.01, 0, 0, 1.0]]), (sizes[0], 1)))      # equal points
    flat = np.concatenate([rng.uniform(-0.2, 0.2, (sizes[0], 3)), rng.normal(size=(sizes[0], 3))], 1)
    flat[:, 2] = 0.125                                                                   # a plane
    pts.append(flat)
    n = [len(p) for p in pts]
    lib = I.ShapeLibrary(np.concatenate(pts).astype(np.float32), np.concatenate([[0], np.cumsum(n)]).astype(np.int64),
                         np.full(len(n), np.nan, np.float32))
    sa, sb = rng.integers(0, len(n), n_pairs), rng.integers(0, len(n), n_pairs)
    ta, qa, tb, qb = I.overlapping_pair_poses(rng, lib, sa, sb)
    tb[::9], qb[::9] = ta[::9], qa[::9]      # one inside the other's box
    tb[4::9] = ta[4::9] + np.float32(3.0)    # no common box
    return I._pack_pair_scene(lib, ta, qa, tb, qb, sa.astype(np.int32), sb.astype(np.int32),
                              I._interleave_pairs(rng, n_pairs))


@pytest.mark.parametrize("sizes,n_pairs,K", [((1025, 1087, 1088, 1089, 1152), 90, 64),
                                             ((2049, 4097, 1024, 16384), 60, 256),
                                             ((513, 575, 640, 1024, 512), 4100, 32)])
def test_clusters_match_oracle(torch, sizes, n_pairs, K):
    scene = _scene(sizes, n_pairs, 11)
    weights = I.flatten_weights(I.gaussian_weights(I.SMALL_WIDTHS, seed=6, bias_std=0.1))
    ctx = B.context_for_scene(scene, K, WD, weights, precision="bf16")
    objs, pairs = B.scene_tensors(scene)
    idx, counts = (t.cpu().numpy() for t in ctx.debug_crop(objs, pairs))
    rows = np.arange(n_pairs) if n_pairs <= 100 else np.r_[0:40, n_pairs - 40:n_pairs]
    sub = scene.pairs[rows]
    _, ridx, rcounts = O.crop(scene.lib.pts, scene.lib.offsets, scene.pos, scene.quat, scene.shape, sub, K)
    assert (rcounts == 0).any() and (rcounts > K).any() and ((rcounts > 0) & (rcounts < K)).any()
    np.testing.assert_array_equal(counts[rows], rcounts)
    np.testing.assert_array_equal(idx[rows], ridx)
    with_counts, _ = ctx.detect(objs, pairs)
    without, _ = ctx.detect(objs, pairs, want_counts=False)
    np.testing.assert_array_equal(without.cpu().numpy(), with_counts.cpu().numpy())
    ctx.close()


def test_library_memory(torch):
    """A stored point takes 24 bytes on the device, its share of the clusters 15 more, and a row of 32 for gathers where
    all rows are less than a 128th of the free memory: past that the contacts are the same bits without them."""
    rng = np.random.default_rng(3)
    n, half = 16384, rng.uniform(0.05, 0.3, (12, 1, 3))
    pts = np.concatenate([rng.uniform(-half, half, (12, n, 3)), rng.normal(size=(12, n, 3))], 2).astype(np.float32)
    lib = I.ShapeLibrary(pts.reshape(-1, 6), np.arange(13, dtype=np.int64) * n, np.full(12, np.nan, np.float32))
    sa, sb = rng.integers(0, 12, 2100), rng.integers(0, 12, 2100)   # past the batches whose set-up is the crop's own
    scene = I._pack_pair_scene(lib, *I.overlapping_pair_poses(rng, lib, sa, sb), sa.astype(np.int32),
                               sb.astype(np.int32), I._interleave_pairs(rng, 2100))
    weights = I.flatten_weights(I.gaussian_weights(I.SMALL_WIDTHS, seed=6, bias_std=0.1))
    objs, pairs = B.scene_tensors(scene)
    ctx = B.Context(64, WD, 0.01, "fp32")
    ctx.upload_weights(weights)

    def upload(copies):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        ctx.upload_shapes(np.arange(12 * copies + 1, dtype=np.int64) * n, np.tile(lib.pts, (copies, 1)))
        per_point = (free - torch.cuda.mem_get_info()[0]) / (12 * copies * n)
        got = [t.cpu().numpy() for t in (*ctx.detect(objs, pairs), *ctx.detect(objs, pairs[:60].contiguous()),
                                         ctx.pose_gradients(objs, pairs)[0])]
        print(f"{12 * copies * n} points: {per_point:.1f} bytes a point", flush=True)
        return per_point, got

    ctx.reserve(2100)
    _, small = upload(1)
    ctx.upload_shapes(np.array([0, 1], np.int64), lib.pts[:1])   # gives the memory back
    copies = int(torch.cuda.mem_get_info()[0] / 128 / 32 / (12 * n) * 1.03)
    per_point, large = upload(copies)
    assert per_point < 39.2
    ctx.close()
    for a, b in zip(small, large):
        np.testing.assert_array_equal(a, b)
