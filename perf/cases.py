"""The work a user of this library has it do, as measurable cases.

One case is one call (or one burst or epoch of calls) through the public binding on synthetic inputs of the
kind `paper_2304_09439_amd.inputs` draws: object pairs whose world boxes overlap, procedural shapes of 1,024 to
4,096 surface points, He-initialised networks of the two compiled width sets.  `listed()` names the sizes of the
repository's own workloads, `draw()` gives others of the same ranges.
"""

from __future__ import annotations

import functools
import math
import time

import numpy as np
import torch

from paper_2304_09439_amd import binding as B
from paper_2304_09439_amd import inputs as I

PAD = 0.01
NETS = {"small": I.SMALL_WIDTHS, "scale": I.SCALE_WIDTHS}
ENV_SIDE = 0.747        # side of the cube an environment's objects lie in: about 49 pairs per environment
ENV_MAX_OBJECTS = 40
ENV_PAIR_ROOM = 64      # pair capacity per environment of the captured step
TRAIN_BATCHES = 4       # steps of one training pass


def listed():
    return [
        # the smallest request a server or a planner sends: a handful of pairs, all latency
        dict(name="detect_bf16_request", kind="detect", precision="bf16", net="scale", K=128, points=4096, shapes=128,
             pairs=8, counts=False),
        # one small scene in full precision with member counts, the library's plain path
        dict(name="detect_fp32_small", kind="detect", precision="fp32", net="small", K=64, points=1024, shapes=160,
             pairs=80, counts=True),
        # a ragged batch: odd pair count, odd shape size, a K off the powers of two, counts wanted
        dict(name="detect_bf16_ragged", kind="detect", precision="bf16", net="scale", K=96, points=777, shapes=24,
             pairs=1061, counts=True),
        # the at-scale batch in the three precisions that are used in earnest
        dict(name="detect_fp32_scale", kind="detect", precision="fp32", net="scale", K=128, points=2048, shapes=32,
             pairs=16384, counts=False),
        dict(name="detect_bf16_scale", kind="detect", precision="bf16", net="scale", K=128, points=2048, shapes=32,
             pairs=16384, counts=False),
        dict(name="detect_fp8_scale", kind="detect", precision="fp8_encoder", net="scale", K=128, points=2048,
             shapes=32, pairs=16384, counts=False),
        # a vectorised simulation's step: broad phase and detect over every environment, one captured graph
        dict(name="step_bf16_envs", kind="step", precision="bf16", net="scale", K=128, points=2048, shapes=32,
             envs=4096),
        # collision resolution: the logit's gradient with respect to both poses of every pair
        dict(name="pose_grad_fp32", kind="pose_grad", precision="fp32", net="scale", K=128, points=2048, shapes=32,
             pairs=16384),
        # fitting: a few optimiser steps on labelled sphere pairs, then the weights
        dict(name="train_fp32", kind="train", net="small", K=64, points=1024, shapes=32, pairs=4096),
        # the voxel-embedding variant: pairs against resident embeddings, and the embedding of a shape library
        dict(name="voxel_detect", kind="voxel_detect", points=2048, shapes=32, pairs=16384),
        dict(name="voxel_encode", kind="voxel_encode", points=2048, shapes=32),
        # a burst of simulation-step requests (8 to 2,000 pairs each) through the continuous-batching server
        dict(name="serve_bf16_burst", kind="serve", precision="bf16", net="scale", K=128, points=4096, shapes=128,
             envs=256, requests=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["detect"] * 5 + ["step", "pose_grad", "train", "voxel_detect", "voxel_encode", "serve"])
    points, shapes = _log_int(rng, 256, 4096), rng.randint(8, 64)
    if kind == "detect":
        return dict(kind=kind, precision=rng.choice(["fp32", "bf16", "fp8", "fp8_encoder"]),
                    net=rng.choice(["small", "scale", "scale"]), K=32 * rng.randint(1, 4), points=points,
                    shapes=shapes, pairs=_log_int(rng, 1, 16384), counts=rng.random() < 0.3)
    if kind == "step":
        return dict(kind=kind, precision="bf16", net="scale", K=128, points=points, shapes=shapes,
                    envs=_log_int(rng, 16, 4096))
    if kind == "pose_grad":
        return dict(kind=kind, precision=rng.choice(["fp32", "bf16"]), net=rng.choice(["small", "scale"]),
                    K=32 * rng.randint(1, 4), points=points, shapes=shapes, pairs=_log_int(rng, 8, 16384))
    if kind == "train":
        return dict(kind=kind, net=rng.choice(["small", "small", "scale"]), K=32 * rng.randint(1, 4),
                    points=min(points, 2048), shapes=shapes, pairs=_log_int(rng, 64, 4096))
    if kind == "voxel_detect":
        return dict(kind=kind, points=points, shapes=shapes, pairs=_log_int(rng, 1, 16384))
    if kind == "voxel_encode":
        return dict(kind=kind, points=min(points, 2048), shapes=_log_int(rng, 1, 32))
    return dict(kind=kind, precision=rng.choice(["bf16", "fp32"]), net="scale", K=128, points=points, shapes=shapes,
                envs=256, requests=_log_int(rng, 1, 64))


# --------------------------------------------------------------------- inputs

@functools.lru_cache(maxsize=8)
def _library(shapes, points):
    """The object set a program works with: unions of 3-6 ellipsoids and boxes."""
    return I.shape_library(np.random.default_rng([11, shapes, points]), shapes, points, (3, 6), 0.5)


@functools.lru_cache(maxsize=8)
def _spheres(shapes, points):
    return I.sphere_library(np.random.default_rng([12, shapes, points]), shapes, points)


@functools.lru_cache(maxsize=4)
def _weights(net):
    return I.flatten_weights(I.gaussian_weights(NETS[net], seed=0))


@functools.lru_cache(maxsize=1)
def _voxel_weights():
    return I.flatten_weights(I.voxel_weights(seed=0))


def _rotation(q):
    """Rotation matrices [n, 3, 3] of quaternions (w, x, y, z) as given, float64, every product rounded."""
    w, x, y, z = q.double().unbind(-1)
    xx, yy, zz, xy, xz, yz, wx, wy, wz = x * x, y * y, z * z, x * y, x * z, y * z, w * x, w * y, w * z
    return torch.stack([1 - 2 * (yy + zz), 2 * (xy - wz), 2 * (xz + wy), 2 * (xy + wz), 1 - 2 * (xx + zz),
                        2 * (yz - wx), 2 * (xz - wy), 2 * (yz + wx), 1 - 2 * (xx + yy)], -1).reshape(-1, 3, 3)


def _world_extents(lib, shape, q):
    """Min / max [n, 3] of every object's rotated cloud relative to its origin."""
    R = _rotation(torch.from_numpy(q).cuda())
    lo = torch.empty(len(shape), 3, dtype=torch.float64, device="cuda")
    hi = torch.empty_like(lo)
    ids = torch.from_numpy(shape).cuda()
    for s in range(lib.n_shapes):
        p = torch.from_numpy(lib.shape_points(s)[:, :3]).cuda().double()
        for rows in torch.nonzero(ids == s).flatten().split(1024):
            for k in range(3):
                v = R[rows, k, 0, None] * p[:, 0] + R[rows, k, 1, None] * p[:, 1] + R[rows, k, 2, None] * p[:, 2]
                lo[rows, k], hi[rows, k] = v.amin(1), v.amax(1)
    return lo.cpu().numpy(), hi.cpu().numpy()


def _scene(case, seed):
    """Pairs of library shapes whose world boxes overlap; about half the pairs given in reverse."""
    lib, n = _library(case["shapes"], case["points"]), case["pairs"]
    rng = np.random.default_rng([1, seed])
    shape = rng.integers(0, lib.n_shapes, 2 * n).astype(np.int32)
    quat = I.uniform_quaternions(rng, 2 * n).astype(np.float32)
    pos = rng.uniform(-1.0, 1.0, (2 * n, 3)).astype(np.float32)
    lo, hi = _world_extents(lib, shape, quat)
    pos[1::2] = pos[0::2] + rng.uniform(lo[0::2] - hi[1::2], hi[0::2] - lo[1::2])
    pairs = np.arange(2 * n, dtype=np.int32).reshape(n, 2)
    swap = rng.random(n) < 0.5
    pairs[swap] = pairs[swap][:, ::-1]
    return I.Scene(lib, pos, quat, shape, pairs)


def _train_scene(case, seed):
    """Labelled sphere pairs at centre distances around contact, one scene over all batches."""
    lib, n = _spheres(case["shapes"], case["points"]), case["pairs"] * TRAIN_BATCHES
    rng = np.random.default_rng([2, seed])
    sa, sb = (rng.integers(0, lib.n_shapes, n).astype(np.int32) for _ in range(2))
    ta, qa, tb, qb = I.sphere_pair_poses(rng, lib.radius[sa], lib.radius[sb])
    pairs = np.arange(2 * n, dtype=np.int32).reshape(n, 2)
    swap = rng.random(n) < 0.5
    pairs[swap] = pairs[swap][:, ::-1]
    mix = lambda a, b: np.stack([a, b], 1).reshape((2 * n,) + a.shape[1:])  # noqa: E731
    scene = I.Scene(lib, mix(ta, tb), mix(qa, qb), mix(sa, sb), pairs)
    return scene, I.sphere_labels(scene)["flag"].astype(np.float32)


def _environments(case, seed):
    """1 to 40 objects per environment at random poses in a cube."""
    lib = _library(case["shapes"], case["points"])
    rng = np.random.default_rng([3, seed])
    sizes = rng.integers(1, ENV_MAX_OBJECTS + 1, case["envs"])
    n = int(sizes.sum())
    shape = rng.integers(0, lib.n_shapes, n).astype(np.int32)
    pos = ((rng.random((n, 3)) - 0.5) * ENV_SIDE).astype(np.float32)
    quat = I.uniform_quaternions(rng, n).astype(np.float32)
    offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    return lib, shape, pos, quat, offsets


def _requests(case, seed):
    """Requests of 8 to 2,000 pairs: each moves every object of some environments and asks for their pairs."""
    lib, shape, pos0, quat0, offsets = _environments(case, seed)
    rng = np.random.default_rng([4, seed])
    sizes = np.diff(offsets)
    pos = (pos0 + rng.normal(0.0, 0.002, pos0.shape)).astype(np.float32)
    quat = I.uniform_quaternions(rng, len(shape)).astype(np.float32)
    slices = [(int(k), offsets[:-1][sizes == k].astype(np.int64)) for k in np.unique(sizes)]
    found = I.broad_phase(I._local_boxes(lib), shape, slices, pos.astype(np.float64), quat)
    owner = np.searchsorted(offsets, found[:, 0], side="right") - 1
    by_env = [found[owner == e] for e in range(case["envs"])]
    wanted = np.exp(np.random.default_rng(4).uniform(math.log(8), math.log(2000), case["requests"])).astype(int)
    out = []
    for want in wanted:
        envs, have = [], 0
        for e in rng.permutation(case["envs"]):
            if len(by_env[e]):
                envs.append(e)
                have += len(by_env[e])
            if have >= want:
                break
        ids = np.concatenate([np.arange(offsets[e], offsets[e + 1]) for e in envs]).astype(np.int32)
        pairs = np.concatenate([by_env[e] for e in envs])[:want].astype(np.int32)
        out.append((ids, B.pack_objects(pos[ids], quat[ids], shape[ids]), np.ascontiguousarray(pairs)))
    return lib, shape, pos0, quat0, pos, quat, out


# -------------------------------------------------------------- prepare, run

def _context(case, lib, precision):
    w = NETS[case["net"]]
    ctx = B.Context(case["K"], (w.h1, w.h2, w.hh), PAD, precision)
    ctx.upload_shapes(lib.offsets, lib.pts)
    ctx.upload_weights(_weights(case["net"]))
    return ctx


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("detect", "pose_grad"):
        scene = _scene(case, seed)
        s["ctx"] = _context(case, scene.lib, case["precision"])
        s["objs"], s["pairs"] = B.scene_tensors(scene)
        if case["precision"].startswith("fp8"):
            s["ctx"].calibrate(s["objs"], s["pairs"][:1024])
        s["ctx"].reserve(case["pairs"])
        dev = s["objs"].device
        if kind == "detect":
            s["out"] = torch.zeros((case["pairs"], 8), dtype=torch.float32, device=dev)
            s["counts"] = torch.zeros((case["pairs"], 2), dtype=torch.int32, device=dev) if case["counts"] else None
        else:
            s["grad"] = torch.zeros((case["pairs"], 14), dtype=torch.float32, device=dev)
    elif kind == "step":
        lib, shape, pos, quat, offsets = _environments(case, seed)
        s["ctx"] = _context(case, lib, case["precision"])
        cap = ENV_PAIR_ROOM * case["envs"]
        dev = "cuda"
        s["objs"] = torch.from_numpy(B.pack_objects(pos, quat, shape)).to(dev)
        s["pairs"] = torch.zeros((cap, 2), dtype=torch.int32, device=dev)
        s["count"] = torch.zeros(2, dtype=torch.int32, device=dev)
        s["out"] = torch.zeros((cap, 8), dtype=torch.float32, device=dev)
        s["graph"] = s["ctx"].capture_step_graph(s["objs"], torch.from_numpy(offsets).to(dev), s["pairs"], s["count"],
                                                 s["out"])
    elif kind == "train":
        scene, labels = _train_scene(case, seed)
        s["ctx"] = _context(case, scene.lib, "fp32")
        s["objs"], s["pairs"] = B.scene_tensors(scene)
        s["labels"] = torch.from_numpy(labels).to(s["objs"].device)
        s["loss"] = torch.zeros((TRAIN_BATCHES, 2), dtype=torch.float32, device=s["objs"].device)
    elif kind in ("voxel_detect", "voxel_encode"):
        s["ctx"] = B.VoxelContext()
        s["ctx"].upload_weights(_voxel_weights())
        if kind == "voxel_detect":
            scene = _scene(case, seed)
            s["ctx"].upload_shapes(scene.lib.offsets, scene.lib.pts)
            s["objs"], s["pairs"] = B.scene_tensors(scene)
            s["out"] = torch.zeros((case["pairs"], 2), dtype=torch.float32, device=s["objs"].device)
        else:
            s["offsets"], s["points"] = _voxel_library(case, seed)
    else:
        lib, shape, pos0, quat0, _, _, reqs = _requests(case, seed)
        s["ctx"] = _context(case, lib, case["precision"])
        s["srv"] = B.Server(s["ctx"], B.pack_objects(pos0, quat0, shape), slots=3, max_batch_pairs=32768,
                            max_batch_updates=65536, hbm_budget_bytes=8 << 30)
        s["reqs"] = B.Server.pack_requests(reqs)
    return s


def _voxel_library(case, seed):
    """A library of the seed's own: the resident shapes turned and scaled, as a program's own assets differ."""
    lib = _library(case["shapes"], case["points"])
    rng = np.random.default_rng([5, seed])
    pts = lib.pts.copy()
    for s in range(lib.n_shapes):
        rows = slice(lib.offsets[s], lib.offsets[s + 1])
        R = I._scipy_rot(I.uniform_quaternions(rng, 1)[0]).as_matrix()
        scale = rng.uniform(0.5, 1.5)
        pts[rows, :3] = (lib.pts[rows, :3].astype(np.float64) @ R.T) * scale
        pts[rows, 3:] = lib.pts[rows, 3:].astype(np.float64) @ R.T
    return lib.offsets, pts


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "detect":
        return ctx.detect(s["objs"], s["pairs"], s["out"], s["counts"], want_counts=case["counts"])
    if kind == "step":
        s["graph"].launch()
        return s["pairs"], s["count"], s["out"]
    if kind == "pose_grad":
        return ctx.pose_gradients(s["objs"], s["pairs"], s["grad"])[0]
    if kind == "train":
        n = case["pairs"]
        for k in range(TRAIN_BATCHES):
            rows = slice(k * n, (k + 1) * n)
            ctx.train_step(s["objs"], s["pairs"][rows], s["labels"][rows], loss=s["loss"][k])
        return s["loss"], ctx.get_weights(0)
    if kind == "voxel_detect":
        return ctx.detect(s["objs"], s["pairs"], s["out"], want_counts=False)[0]
    if kind == "voxel_encode":
        ctx.upload_shapes(s["offsets"], s["points"])
        return ctx.embeddings()
    srv = s["srv"]
    contacts, counts = [], []
    for rid in srv.submit_many_arrays(*s["reqs"]):
        while (r := srv.poll(rid)) is None:
            time.sleep(20e-6)
        contacts.append(r[0])
        counts.append(r[1])
    return np.concatenate(contacts), np.concatenate(counts)


# ----------------------------------------------------------------------- work

def _row_share(K, points):
    """Share of the 2K encoder rows that are members, about: a crop holds a third of a cloud, or nothing."""
    return 0.87 * min(1.0, 0.36 * points / K)


def _net_flops(net, K, points, pairs):
    w = NETS[net]
    rows = 2 * K * _row_share(K, points)
    return pairs * 2.0 * (rows * (6 * w.h1 + w.h1 * w.h2) + 2 * w.h2 * w.hh + w.hh * w.hh + 8 * w.hh)


VOXEL_PAIR_FLOPS = 2.0 * (2 * (28 * 128 + 2 * 128 * 128) + 3 * 128 * 128 + 128)
# U-Net taps that meet a cell: 6^3 -> 4^3 and back all 27, 4^3 with border (10/4)^3
VOXEL_SHAPE_FLOPS = 2.0 * (64 * 27 * 256 * 128 + 64 * 15.625 * (4 * 128 * 128 + 2 * 256 * 128)
                           + 64 * 27 * 256 * 128 + 216 * 384 * 16)
VOXEL_POINT_FLOPS = 2.0 * (3 * 256 + 2 * 256 * 256)


def work(case):
    kind = case["kind"]
    lib = 24.0 * case["shapes"] * case["points"]
    if kind.startswith("voxel"):
        if kind == "voxel_detect":
            n = case["pairs"]
            return dict(bytes=case["shapes"] * 216 * 64.0 + n * (2 * 32 + 8 + 8.0) + 4 * 87000.0,
                        flops=VOXEL_PAIR_FLOPS * n)
        return dict(bytes=lib + 4 * 5.45e6 + case["shapes"] * 216 * 64.0,
                    flops=case["shapes"] * (VOXEL_SHAPE_FLOPS + case["points"] * VOXEL_POINT_FLOPS))
    weight = {"bf16": 2.0, "fp32": 4.0}.get(case.get("precision", "fp32"), 1.5) * NETS[case["net"]].n_floats()
    if kind == "detect":
        n = case["pairs"]
        return dict(bytes=lib + weight + n * (2 * 32 + 8 + 32 + (8.0 if case["counts"] else 0)),
                    flops=_net_flops(case["net"], case["K"], case["points"], n))
    if kind == "step":
        n = 49.0 * case["envs"]
        return dict(bytes=lib + weight + 20.5 * 32 * case["envs"] + n * (8 + 32),
                    flops=_net_flops(case["net"], case["K"], case["points"], n))
    w = NETS[case["net"]]
    if kind == "pose_grad":
        n = case["pairs"]
        back = 2.0 * (w.hh * w.hh + w.hh * w.h2) + 2.0 * w.h2 * w.h1 * 12
        return dict(bytes=lib + weight + n * (2 * 32 + 8 + 56.0),
                    flops=_net_flops(case["net"], case["K"], case["points"], n) + n * back)
    if kind == "train":
        n = case["pairs"] * TRAIN_BATCHES
        back = 2.0 * (w.hh * w.hh + w.hh * 2 * w.h2) * 2 + 2.0 * (2 * w.h2 * w.h1 * 14)
        return dict(bytes=lib + TRAIN_BATCHES * 7 * weight + n * (2 * 32 + 8 + 4.0),
                    flops=_net_flops(case["net"], case["K"], case["points"], n) + n * back)
    n = 360.0 * case["requests"]
    return dict(bytes=lib + weight + n * (8 + 32 + 8.0) + 150.0 * 32 * case["requests"],
                flops=_net_flops(case["net"], case["K"], case["points"], n))


# ---------------------------------------------------------------------- exact
#
# The path written plainly in 64 bits.  The geometry keeps the order of operations that fixes the crop sets.

def _unpack(flat, widths, dev):
    shapes = [(widths.h1, 6), (widths.h2, widths.h1), (widths.hh, 2 * widths.h2), (widths.hh, widths.hh),
              (8, widths.hh)]
    flat = torch.from_numpy(flat).to(dev).double()
    out, o = [], 0
    for r, c in shapes:
        out += [flat[o:o + r * c].reshape(r, c), flat[o + r * c:o + r * c + r]]
        o += r * c + r
    return out


def _cloud(lib, dev):
    pts = torch.from_numpy(lib.pts).to(dev).double().reshape(lib.n_shapes, -1, 6)
    return pts, pts[:, :, :3].amin(1), pts[:, :, :3].amax(1)


def _relative(pa, qa, pb, qb):
    Ra, Rb = _rotation(qa), _rotation(qb)
    col = lambda i: Ra[:, :, i]  # noqa: E731
    R = torch.stack([torch.stack([(col(i)[:, 0] * Rb[:, 0, j] + col(i)[:, 1] * Rb[:, 1, j]) + col(i)[:, 2] * Rb[:, 2, j]
                                  for j in range(3)], -1) for i in range(3)], 1)
    d = pb - pa
    t = torch.stack([(col(i)[:, 0] * d[:, 0] + col(i)[:, 1] * d[:, 1]) + col(i)[:, 2] * d[:, 2] for i in range(3)], -1)
    return Ra, R, t


def _apply(R, t, p):
    """[n, 3, 3], [n, 3] on [n, m, 3]."""
    return torch.stack([((R[:, i, 0, None] * p[..., 0] + R[:, i, 1, None] * p[..., 1]) + R[:, i, 2, None] * p[..., 2])
                        + t[:, i, None] for i in range(3)], -1)


def _first(member, K):
    """Indices [n, K] of the first K members in stored order, and which of them exist."""
    n, m = member.shape
    key = torch.where(member, torch.arange(m, device=member.device), m)
    key = torch.nn.functional.pad(key, (0, max(0, K - m)), value=m)
    key = key.sort(1).values[:, :K]
    return key.clamp(max=m - 1), key < m


def _crops(cloud, lo, hi, sa, sb, R, t, K):
    """(stored rows [n, K, 6], exist [n, K]) of both objects, selected by the crop box in a's frame."""
    c, e = 0.5 * (lo[sb] + hi[sb]), 0.5 * (hi[sb] - lo[sb])
    cc = _apply(R, t, c[:, None])[:, 0]
    A = R.abs()
    ee = torch.stack([(A[:, i, 0] * e[:, 0] + A[:, i, 1] * e[:, 1]) + A[:, i, 2] * e[:, 2] for i in range(3)], -1)
    blo = torch.maximum(lo[sa], cc - ee) - PAD
    bhi = torch.minimum(hi[sa], cc + ee) + PAD
    out = []
    for stored, at in ((cloud[sa], None), (cloud[sb], (R, t))):
        q = stored[..., :3] if at is None else _apply(*at, stored[..., :3])
        idx, ok = _first(((q >= blo[:, None]) & (q <= bhi[:, None])).all(-1), K)
        out.append((stored.gather(1, idx[..., None].expand(-1, -1, 6)), ok))
    return out


def _encode(rows, ok, W):
    h = torch.relu(torch.relu(rows @ W[0].T + W[1]) @ W[2].T + W[3])
    return torch.where(ok[..., None], h, 0.0).max(1).values


def _features(crops, R, t, W):
    (ra, oka), (rb, okb) = crops
    zero = torch.zeros_like(t)
    moved = torch.cat([_apply(R, t, rb[..., :3]), _apply(R, zero, rb[..., 3:])], -1)
    return torch.cat([_encode(ra, oka, W), _encode(moved, okb, W)], 1)


def _head(z, W):
    return torch.relu(torch.relu(z @ W[4].T + W[5]) @ W[6].T + W[7]) @ W[8].T + W[9]


def _canonical(pairs):
    a, b = pairs.min(1).values, pairs.max(1).values
    return a, b, torch.where(pairs[:, 0] > pairs[:, 1], -1.0, 1.0).double()


def _pair_chunk(case):
    return max(16, min(1024, (1 << 21) // max(case["points"], 2 * case["K"])))


def _contacts(case, lib, pos, quat, shape, pairs):
    dev = "cuda"
    W = _unpack(_weights(case["net"]), NETS[case["net"]], dev)
    cloud, lo, hi = _cloud(lib, dev)
    pos, quat, shape, pairs = (torch.as_tensor(v).to(dev) for v in (pos, quat, shape, pairs))
    pos, shape, pairs = pos.double(), shape.long(), pairs.long()
    out = []
    for pr in pairs.split(_pair_chunk(case)):
        a, b, sgn = _canonical(pr)
        Ra, R, t = _relative(pos[a], quat[a], pos[b], quat[b])
        y = _head(_features(_crops(cloud, lo, hi, shape[a], shape[b], R, t, case["K"]), R, t, W), W)
        point = (Ra @ y[:, 1:4, None])[..., 0] + pos[a]
        normal = sgn[:, None] * (Ra @ y[:, 4:7, None])[..., 0]
        out.append(torch.cat([y[:, :1], point, normal, y[:, 7:]], 1))
    return torch.cat(out)


def _env_pairs(lib, shape, pos, quat, offsets):
    dev = "cuda"
    _, lo, hi = _cloud(lib, dev)
    sh = torch.from_numpy(shape).to(dev).long()
    c, e = 0.5 * (lo + hi)[sh], 0.5 * (hi - lo)[sh]
    R = _rotation(torch.from_numpy(quat).to(dev))
    cw = _apply(R, torch.from_numpy(pos).to(dev).double(), c[:, None])[:, 0]
    A = R.abs()
    ew = torch.stack([(A[:, i, 0] * e[:, 0] + A[:, i, 1] * e[:, 1]) + A[:, i, 2] * e[:, 2] for i in range(3)], -1)
    blo, bhi = cw - ew, cw + ew
    sizes = np.diff(offsets)
    found = []
    for n in np.unique(sizes):
        i, j = np.triu_indices(int(n), 1)
        if len(i) == 0:
            continue
        start = torch.from_numpy(offsets[:-1][sizes == n]).to(dev).long()
        gi = (start[:, None] + torch.from_numpy(i).to(dev)).flatten()
        gj = (start[:, None] + torch.from_numpy(j).to(dev)).flatten()
        hit = ((blo[gi] <= bhi[gj]) & (blo[gj] <= bhi[gi])).all(-1)
        found.append(torch.stack([gi[hit], gj[hit]], 1))
    pairs = torch.cat(found)
    return pairs[(pairs[:, 0] * len(shape) + pairs[:, 1]).argsort()]


def _pose_gradients(case, scene):
    dev = "cuda"
    W = _unpack(_weights(case["net"]), NETS[case["net"]], dev)
    cloud, lo, hi = _cloud(scene.lib, dev)
    pos, quat = torch.from_numpy(scene.pos).to(dev).double(), torch.from_numpy(scene.quat).to(dev).double()
    shape, pairs = torch.from_numpy(scene.shape).to(dev).long(), torch.from_numpy(scene.pairs).to(dev).long()
    out = []
    for pr in pairs.split(_pair_chunk(case) // 4):
        a, b, sgn = _canonical(pr)
        leaf = [v.clone().requires_grad_() for v in (pos[a], quat[a], pos[b], quat[b])]
        _, R, t = _relative(*leaf)
        with torch.no_grad():
            crops = _crops(cloud, lo, hi, shape[a], shape[b], R, t, case["K"])
        _head(_features(crops, R, t, W), W)[:, 0].sum().backward()
        first, second = torch.cat([leaf[0].grad, leaf[1].grad], 1), torch.cat([leaf[2].grad, leaf[3].grad], 1)
        back = (sgn < 0)[:, None]
        out.append(torch.cat([torch.where(back, second, first), torch.where(back, first, second)], 1))
    return torch.cat(out)


def _train(case, scene, labels):
    dev = "cuda"
    widths = NETS[case["net"]]
    flat = torch.from_numpy(_weights(case["net"])).to(dev).double()
    cloud, lo, hi = _cloud(scene.lib, dev)
    pos, quat = torch.from_numpy(scene.pos).to(dev).double(), torch.from_numpy(scene.quat).to(dev)
    shape, pairs = torch.from_numpy(scene.shape).to(dev).long(), torch.from_numpy(scene.pairs).to(dev).long()
    y = torch.from_numpy(labels).to(dev).double()
    n, losses = case["pairs"], []
    m, v = torch.zeros_like(flat), torch.zeros_like(flat)
    for k in range(TRAIN_BATCHES):
        w = flat.clone().requires_grad_()
        loss = torch.zeros(2, dtype=torch.float64, device=dev)
        for at in torch.arange(k * n, (k + 1) * n, device=dev).split(_pair_chunk(case) // 2):
            W, o = [], 0
            for r, c in [(widths.h1, 6), (widths.h2, widths.h1), (widths.hh, 2 * widths.h2), (widths.hh, widths.hh),
                         (8, widths.hh)]:
                W += [w[o:o + r * c].reshape(r, c), w[o + r * c:o + r * c + r]]
                o += r * c + r
            a, b, _ = _canonical(pairs[at])
            _, R, t = _relative(pos[a], quat[a], pos[b], quat[b])
            z = _features(_crops(cloud, lo, hi, shape[a], shape[b], R, t, case["K"]), R, t, W)
            x = _head(z, W)[:, 0]
            bce = (x.clamp(min=0) - x * y[at] + torch.log1p(torch.exp(-x.abs()))).sum() / n
            reg = 0.5 * z.square().sum() / n
            (bce + reg).backward()
            loss += torch.stack([bce.detach(), reg.detach()])
        losses.append(loss)
        g = w.grad
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        flat = flat - 1e-3 * (m / (1 - 0.9 ** (k + 1))) / ((v / (1 - 0.999 ** (k + 1))).sqrt() + 1e-8)
    return torch.stack(losses), flat


def _voxel_unpack(dev):
    flat, out, o = torch.from_numpy(_voxel_weights()).to(dev).double(), [], 0
    for wshape, nb in I.VOXEL_LAYERS:
        n = int(np.prod(wshape))
        out += [flat[o:o + n].reshape(wshape), flat[o + n:o + n + nb]]
        o += n + nb
    return out


def _conv(x, W, b, pad, transposed):
    """3x3x3 convolution (or its transpose) of x [S, C, D, D, D], a matrix product per tap."""
    q = 2 - pad if transposed else pad
    out = x.shape[2] + 2 * q - 2
    x = torch.nn.functional.pad(x, (q,) * 6)
    y = b[:, None] + torch.zeros(x.shape[0], len(b), out ** 3, dtype=x.dtype, device=x.device)
    for u in range(27):
        u0, u1, u2 = ((2 - u // 9, 2 - u // 3 % 3, 2 - u % 3) if transposed else (u // 9, u // 3 % 3, u % 3))
        tap = x[:, :, u0:u0 + out, u1:u1 + out, u2:u2 + out].reshape(x.shape[0], x.shape[1], -1).contiguous()
        y = y + torch.matmul(W[:, :, u // 9, u // 3 % 3, u % 3].contiguous(), tap)
    return torch.relu(y).reshape(x.shape[0], len(b), out, out, out)


def _embeddings(offsets, pts):
    dev = "cuda"
    w = _voxel_unpack(dev)
    S = len(offsets) - 1
    xyz = torch.from_numpy(np.ascontiguousarray(pts[:, :3])).to(dev).double().reshape(S, -1, 3)
    lo, hi = xyz.amin(1, keepdim=True), xyz.amax(1, keepdim=True)
    cell = (((xyz - lo) * 6.0) / (hi - lo)).floor().clamp(max=5).long()
    cell = (cell[..., 0] * 6 + cell[..., 1]) * 6 + cell[..., 2]
    h = xyz
    for k in range(3):
        h = torch.relu(h @ w[2 * k].T + w[2 * k + 1])
    grid = torch.zeros(S, 216, 256, dtype=torch.float64, device=dev)
    grid = grid.scatter_reduce(1, cell[..., None].expand(-1, -1, 256), h, "amax")
    x = grid.transpose(1, 2).reshape(S, 256, 6, 6, 6).contiguous()
    c = []
    for k in range(4):
        x = _conv(x, w[6 + 2 * k], w[7 + 2 * k], 0 if k == 0 else 1, False)
        c.append(x)
    g = torch.cat([x.flatten(2).amax(2), x.flatten(2).mean(2)], 1)
    for k in range(4):
        x = _conv(x if k == 0 else torch.cat([x, c[3 - k]], 1), w[14 + 2 * k], w[15 + 2 * k], 0 if k == 3 else 1, True)
    rows = torch.cat([x.flatten(2).transpose(1, 2), g[:, None].expand(-1, 216, -1)], 2)
    return rows @ w[22].T + w[23]


def _voxel_pairs(scene):
    dev = "cuda"
    w = _voxel_unpack(dev)
    emb = _embeddings(scene.lib.offsets, scene.lib.pts)
    _, lo, hi = _cloud(scene.lib, dev)
    pos, quat = torch.from_numpy(scene.pos).to(dev).double(), torch.from_numpy(scene.quat).to(dev)
    shape, pairs = torch.from_numpy(scene.shape).to(dev).long(), torch.from_numpy(scene.pairs).to(dev).long()
    step = (hi - lo) / 6.0
    eps = ((step[:, 0] * step[:, 0] + step[:, 1] * step[:, 1]) + step[:, 2] * step[:, 2]).sqrt() * 0.5
    i = torch.arange(216, device=dev)
    ijk = torch.stack([i // 36, i // 6 % 6, i % 6], -1).double()
    centres = lo[:, None] + (ijk + 0.5) * step[:, None]
    out = []
    for pr in pairs.split(2048):
        a, b, _ = _canonical(pr)
        sa, sb = shape[a], shape[b]
        _, R, t = _relative(pos[a], quat[a], pos[b], quat[b])
        d = centres[sa] - t[:, None]
        xa = torch.stack([(R[:, 0, k, None] * d[..., 0] + R[:, 1, k, None] * d[..., 1]) + R[:, 2, k, None] * d[..., 2]
                          for k in range(3)], -1)
        xb = _apply(R, t, centres[sb])
        pooled = []
        for x, own, other in ((xa, sa, sb), (xb, sb, sa)):
            e = eps[own][:, None, None]
            sel = ((x >= lo[other][:, None] - e) & (x <= hi[other][:, None] + e)).all(-1).double()
            pooled.append(torch.matmul(sel[:, None], emb[own])[:, 0] / sel.sum(1, keepdim=True).clamp(min=1))
        ta = -torch.stack([(R[:, 0, k] * t[:, 0] + R[:, 1, k] * t[:, 1]) + R[:, 2, k] * t[:, 2] for k in range(3)], -1)
        za = torch.cat([pooled[0], ta, R.transpose(1, 2).reshape(-1, 9)], 1)
        zb = torch.cat([pooled[1], t, R.reshape(-1, 9)], 1)
        for k in (24, 26, 28):
            za, zb = torch.relu(za @ w[k].T + w[k + 1]), torch.relu(zb @ w[k].T + w[k + 1])
        g = torch.maximum(za, zb)
        for k in (30, 32, 34):
            g = torch.relu(g @ w[k].T + w[k + 1])
        logit = g @ w[36].T + w[37]
        out.append(torch.cat([logit, torch.sigmoid(logit)], 1))
    return torch.cat(out)


def exact(case, seed):
    kind = case["kind"]
    if kind == "detect":
        sc = _scene(case, seed)
        return _contacts(case, sc.lib, sc.pos, sc.quat, sc.shape, sc.pairs), None
    if kind == "step":
        lib, shape, pos, quat, offsets = _environments(case, seed)
        pairs = _env_pairs(lib, shape, pos, quat, offsets)[:ENV_PAIR_ROOM * case["envs"]]
        out = torch.zeros((ENV_PAIR_ROOM * case["envs"], 8), dtype=torch.float64, device="cuda")
        out[:len(pairs)] = _contacts(case, lib, pos, quat, shape, pairs)
        return None, None, out
    if kind == "pose_grad":
        return _pose_gradients(case, _scene(case, seed))
    if kind == "train":
        return _train(case, *_train_scene(case, seed))
    if kind == "voxel_detect":
        return _voxel_pairs(_scene(case, seed))
    if kind == "voxel_encode":
        return _embeddings(*_voxel_library(case, seed))
    lib, shape, _, _, pos, quat, reqs = _requests(case, seed)
    return _contacts(case, lib, pos, quat, shape, np.concatenate([r[2] for r in reqs])), None
