"""Performance cases of the framework: what its users have it do, through its public entry points.

A user decimates meshes (one scan, a mini-batch of rooms, a ladder of resolutions), builds the index
arrays of the convolutions for them, pools and unpools features over the recorded clusters, and runs
the mesh convolutions forward (inference) or forward and backward (training).  Sizes: lattices and
synthetic rooms from 4 thousand vertices (a small object) over 115 thousand (a scanned room) to 1.2
million (a large scan), single lattices up to 10 million; 3 to 300 feature channels, up to 13 Gaussian
components.  A case is a dict of plain values; see ``listed`` for what each stands for.
"""
import functools
import math

import numpy as np
import torch

import paper_2103_15076_amd as pk
from paper_2103_15076_amd import meshgen

DEV = "cuda:0"


def _decimate(shape, verts, keep, meshes=1, levels=1, placement="mean", absorb=False, shuffle=False):
    return dict(op="decimate", shape=shape, verts=verts, keep=keep, meshes=meshes, levels=levels, placement=placement,
                absorb=absorb, shuffle=shuffle)


def _conv(op, verts, meshes, channels, components, learn=False):
    return dict(op=op, shape="room", verts=verts, meshes=meshes, channels=channels, components=components, learn=learn)


def listed():
    return [
        # the smallest mesh of the benchmark: launches and waits count, not bytes
        dict(_decimate("lattice", 4096, 0.25), name="decimate-lattice-4k"),
        # the headline workload: one scanned room to 36 % of its vertices
        dict(_decimate("room", 115000, 0.361), name="decimate-room-115k"),
        # the largest scan of the paper's datasets
        dict(_decimate("room", 1200000, 0.25), name="decimate-scene-1.2m"),
        # a network's mini-batch: 16 rooms, the four resolutions of its encoder in a row
        dict(_decimate("room", 60000, 0.4, meshes=16, levels=4), name="decimate-ladder-16x60k"),
        # training-time augmentation: seeded shuffle of equal-cost pairs, leftover vertices absorbed (Alg. 2 line 11)
        dict(_decimate("room", 20000, 0.4, meshes=8, absorb=True, shuffle=True), name="decimate-augment-8x20k"),
        # beyond scans: one lattice of 10 million vertices / 20 million facets
        dict(_decimate("lattice", 10240000, 0.25), name="decimate-lattice-10m"),
        # a pooling layer of a training step over one room's clusters: member lists, max pooling and
        # unpooling, forward and backward
        dict(op="pool", shape="room", verts=115000, keep=0.361, channels=64, mode="max", name="pool-train-115k"),
        # index arrays, normals, levels and fuzzy coefficients of a new mini-batch (once per step: its meshes are new)
        dict(_conv("setup", 60000, 16, 0, 6), name="conv-setup-16x60k"),
        # inference on one room: vertex2facet and facet2vertex at an inner layer's width
        dict(_conv("forward", 115000, 1, 64, 6), name="conv-forward-115k"),
        # a training step's convolution on the mini-batch, fixed Gaussian components
        dict(_conv("train", 60000, 16, 64, 6), name="conv-train-16x60k"),
        # the first layer of a network in training: few, odd-sized channels (position and colour), components learnt
        dict(_conv("train", 60000, 1, 6, 6, learn=True), name="conv-train-60k-c6"),
        # facet2facet on a textured room in training: 8 texture points per facet on average
        dict(op="texture", shape="room", verts=115000, points=8, channels=32, name="texture-train-115k"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A channel count: of inner layers (multiples of 8) more often than of first layers and heads (any)."""
    c = _log(rng, lo, hi)
    return max(8, c // 8 * 8) if rng.random() < 0.6 else c


def draw(rng):
    """One more case: sizes over the logarithm of the ranges above, options as often as they are used."""
    kind = rng.choice(("single", "single", "lattice", "batch", "pool", "setup", "forward", "train", "train", "texture"))
    options = dict(placement="inverse" if rng.random() < 0.15 else "mean", absorb=rng.random() < 0.15,
                   shuffle=rng.random() < 0.15)
    keep = round(rng.uniform(0.1, 0.7), 3)
    if kind == "single":
        return _decimate("room", _log(rng, 9000, 1200000), keep, **options)
    if kind == "lattice":
        return _decimate("lattice", _log(rng, 4000, 10000000), keep, **options)
    if kind == "batch":
        meshes = rng.randint(2, 16)
        return _decimate("room", _log(rng, 4000, 1000000 // meshes), keep, meshes=meshes, levels=rng.randint(1, 4),
                         **options)
    if kind == "pool":
        channels = _width(rng, 1, 256)
        return dict(op="pool", shape="room", verts=_log(rng, 5000, min(1200000, 60000000 // channels)), keep=keep,
                    channels=channels, mode=rng.choice(("max", "avg", "weighted")))
    if kind == "texture":
        channels, points = _width(rng, 3, 64), rng.randint(1, 16)
        return dict(op="texture", shape="room", verts=_log(rng, 5000, min(400000, 60000000 // (2 * points * channels))),
                    points=points, channels=channels)
    meshes = rng.choice((1, 1, rng.randint(2, 16)))
    channels = 0 if kind == "setup" else _width(rng, 3, 300)
    total = _log(rng, 5000 * meshes, min(960000, 60000000 // max(channels, 1)))
    return _conv(kind, total // meshes, meshes, channels, rng.randint(1, 13), learn=kind == "train" and rng.random() < 0.4)


# ---- inputs -----------------------------------------------------------------------------------


def _lattice(n, gen):
    """Height field like meshgen.noisy_grid, made on the GPU: about n vertices, split cells."""
    w = max(2, int(math.sqrt(n)))
    h = max(2, n // w)
    x = torch.linspace(0, 1, w, device=DEV, dtype=torch.float64)
    y = torch.linspace(0, 1, h, device=DEV, dtype=torch.float64)
    z = 0.05 * torch.outer(torch.cos(6 * y), torch.sin(6 * x))
    z = z + torch.randn((h, w), generator=gen, device=DEV, dtype=torch.float32) * (0.128 / max(w, h))
    verts = torch.stack([x.expand(h, w), y[:, None].expand(h, w), z], dim=2).to(torch.float32).reshape(-1, 3)
    v00 = (torch.arange(h - 1, device=DEV, dtype=torch.int32)[:, None] * w + torch.arange(w - 1, device=DEV, dtype=torch.int32)).reshape(-1)
    facets = torch.stack([v00, v00 + 1, v00 + w + 1, v00, v00 + w + 1, v00 + w], dim=1).reshape(-1, 3)
    return verts.contiguous(), facets.contiguous()


@functools.lru_cache(maxsize=2)
def _rooms(verts, meshes):
    """Surfaces of the rooms without their measurement noise: (verts, facets, nv per mesh, nf per mesh).  The
    rooms' furniture goes by the case, so that sizes do; the noise goes by the seed."""
    large = verts > 400000
    parts = [meshgen.room_scene_sized(1000 * meshes + k, verts, room=(30.0, 20.0, 3.0) if large else (10.0, 8.0, 3.0),
                                      n_boxes=300 if large else 40, jitter=0.0) for k in range(meshes)]
    nv, nf = [p[0].shape[0] for p in parts], [p[1].shape[0] for p in parts]
    base = np.concatenate([[0], np.cumsum(nv)])
    return (np.concatenate([p[0] for p in parts]), np.concatenate([p[1] + np.int32(base[k]) for k, p in enumerate(parts)]),
            nv, nf)


def _meshes(case, gen):
    """(verts, facets, nv per mesh, nf per mesh) of the case, vertices and facets on the GPU."""
    if case["shape"] == "lattice":
        v, f = _lattice(case["verts"], gen)
        return v, f, [v.shape[0]], [f.shape[0]]
    v, f, nv, nf = _rooms(case["verts"], case.get("meshes", 1))
    v = torch.from_numpy(v).to(DEV)
    return v + torch.randn(v.shape, generator=gen, device=DEV) * 0.003, torch.from_numpy(f).to(DEV), nv, nf


def _targets(nv, keep, levels):
    """Vertex budget of every mesh at every level (256 at least, as the paper's smallest)."""
    out, now = [], list(nv)
    for _ in range(levels):
        now = [max(min(n, 256), int(n * keep)) for n in now]
        out.append(now)
    return out


def prepare(case, seed):
    torch.cuda.set_device(0)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def randn(*shape, scale=1.0):
        return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32) * scale

    v, f, nv, nf = _meshes(case, gen)
    n, m = v.shape[0], f.shape[0]
    ctx = pk.Context(n, m, len(nv), device=0)
    s = dict(case=case, ctx=ctx, verts=v, facets=f, nv=nv, nf=nf)
    op, c = case["op"], case.get("channels", 0)
    if op == "decimate":
        if case["placement"] == "inverse":
            ctx.set_placement(pk.PICASSO_PLACE_INVERSE)
        ctx.set_option(pk.PICASSO_OPT_ABSORB, int(case["absorb"]))
        ctx.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, seed + 1 if case["shuffle"] else 0)
        s["targets"] = _targets(nv, case["keep"], case["levels"])
        # the program's buffers for each level's mesh and clustering (rows beyond the counts stay as they are)
        s["buffers"] = [(torch.zeros((n, 3), device=DEV), torch.zeros((m, 3), dtype=torch.int32, device=DEV),
                         torch.zeros((n,), dtype=torch.int32, device=DEV)) for _ in range(case["levels"])]
    elif op == "pool":
        _, vo, _, cid = ctx.picasso_decimate(v, f, max(1, int(n * case["keep"])))
        s.update(cid=cid, n_out=vo.shape[0], x=randn(n, c), gy=randn(vo.shape[0], c), y=randn(vo.shape[0], c), gx=randn(n, c),
                 mode={"max": pk.PICASSO_POOL_MAX, "avg": pk.PICASSO_POOL_AVG, "weighted": pk.PICASSO_POOL_WEIGHTED}[case["mode"]],
                 weight=torch.rand((n,), generator=gen, device=DEV) if case["mode"] == "weighted" else None)
    elif op == "texture":
        p = case["points"] * m  # ... of which a facet holds anything from none to a few times the average
        poff = torch.randint(0, p + 1, (m + 1,), generator=gen, device=DEV, dtype=torch.int32).sort().values
        poff[0], poff[m] = 0, p
        bary = -torch.log(1.0 - torch.rand((p, 3), generator=gen, device=DEV))
        bary = (bary / bary.sum(1, keepdim=True)).contiguous()
        s.update(poff=poff, bary=bary, tex=randn(p, c), w=randn(3, c, scale=0.3), gy=randn(m, c))
    else:
        t = case["components"]
        mu = randn(t, 3)
        s.update(mu=(mu / mu.norm(dim=1, keepdim=True)).contiguous(), inv_var=torch.full((t,), 2.0, device=DEV))
        if op != "setup":
            s["off"], s["cor"] = ctx.picasso_vertex_corner_csr(f, n)
            normals, _, s["level"] = ctx.picasso_facet_geometry(v, f, nf=nf)
            s["pi"] = ctx.picasso_fuzzy_coefficients(normals, s["mu"], s["inv_var"])
            s.update(x=randn(n, c), w3=randn(3, c, scale=0.3), wt=randn(t, c, scale=0.3), g=randn(n, c))
    return s


def run(s):
    case, ctx, op = s["case"], s["ctx"], s["case"]["op"]
    if op == "decimate":
        out, v, f, nv, nf = [], s["verts"], s["facets"], s["nv"], s["nf"]
        if len(nv) == 1 and case["levels"] == 1:
            st, vo, fo, _ = ctx.picasso_decimate(v, f, s["targets"][0][0], *s["buffers"][0])
            return st, vo.shape[0], fo.shape[0], s["buffers"][0]
        for target, buffers in zip(s["targets"], s["buffers"]):
            st, v, f, _, nv, nf = ctx.picasso_decimate_batch(v, f, nv, nf, target, *buffers)
            out.append((st, nv, nf, buffers))
        return out
    if op == "pool":
        mode, w = s["mode"], s["weight"]
        off, mem = ctx.picasso_cluster_csr(s["cid"], s["n_out"])
        y = ctx.picasso_pool_forward(mode, s["x"], off, mem, weight=w)
        y, arg = y if isinstance(y, tuple) else (y, None)
        gx = ctx.picasso_pool_backward(mode, s["gy"], s["cid"], off, mem, weight=w, argmax=arg)
        up = ctx.picasso_unpool_forward(s["y"], s["cid"])
        return off, mem, y, arg, gx, up, ctx.picasso_unpool_backward(s["gx"], off, mem)
    if op == "texture":
        y = ctx.picasso_f2f_forward(s["tex"], s["bary"], s["poff"], s["w"])
        return y, ctx.picasso_f2f_backward(s["gy"], s["tex"], s["bary"], s["poff"], s["w"])
    if op == "setup":
        off, cor = ctx.picasso_vertex_corner_csr(s["facets"], s["verts"].shape[0])
        normals, area, level = ctx.picasso_facet_geometry(s["verts"], s["facets"], nf=s["nf"])
        return off, cor, normals, area, level, ctx.picasso_fuzzy_coefficients(normals, s["mu"], s["inv_var"])
    n, f = s["x"].shape[0], s["facets"]
    y = ctx.picasso_v2f_forward(s["x"], f, s["level"], s["w3"])
    x2 = ctx.picasso_f2v_forward(y, s["pi"], s["wt"], s["off"], s["cor"], n)
    if op == "forward":
        return y, x2
    gy, gwt, gpi = ctx.picasso_f2v_backward(s["g"], y, s["pi"], s["wt"], f, s["off"], want_gpi=case["learn"])
    gx, gw3 = ctx.picasso_v2f_backward(gy, s["x"], f, s["level"], s["w3"], s["off"], s["cor"])
    return y, x2, gy, gwt, gpi, gx, gw3


# ---- what a pass cannot do without --------------------------------------------------------------


def work(case):
    """Inputs read once, outputs written once; arithmetic of the definitions (a mesh of n vertices has
    about 2 n facets and 3 n edges)."""
    op, n = case["op"], case["verts"] * case.get("meshes", 1)
    c, f = case.get("channels", 0), 2 * n
    if op == "decimate":
        nbytes = flops = 0
        for _ in range(case["levels"]):
            n_out = n * case["keep"]
            nbytes += 12 * n + 12 * 2 * n + 4 * n + 12 * n_out + 12 * 2 * n_out
            # quadrics: a plane per facet, ten sums per corner; a cost (45) per edge of every round, the rounds halving
            flops += 2 * n * 60 + 6 * n * 10 + 45 * 3 * n * 2 * (1 - case["keep"])
            n = n_out
        return dict(bytes=nbytes, flops=flops)
    if op == "pool":
        n_out = n * case["keep"]
        arg = 4 * c * n_out if case["mode"] == "max" else 0
        # member lists; x -> y (+ argmax); gy -> gx; y -> x; gx -> gy
        return dict(bytes=3 * 4 * n + 4 * (4 * c * (n + n_out) + 4 * n) + 2 * arg, flops=4 * c * n)
    if op == "texture":
        p = f * case["points"]
        fwd, bwd = 4 * c * (p + f) + 12 * p + 4 * f, 4 * c * (2 * p + f) + 12 * p + 4 * f
        return dict(bytes=fwd + bwd, flops=p * c * (7 + 8 + 6))
    t = case["components"]
    if op == "setup":
        return dict(bytes=12 * f + 4 * n + 12 * f + 12 * f + 12 * n + 20 * f + 12 * f + 4 * t * f, flops=f * (60 + 20 * t))
    v2f, f2v = 4 * c * (n + f) + 16 * f, 4 * c * (n + f) + 12 * f + 4 * n + 4 * t * f
    nbytes, flops = v2f + f2v, f * c * (14 + 2 * t + 6)
    if op == "train":
        learn = 4 * t * f if case["learn"] else 0
        nbytes += 4 * c * (n + 2 * f) + 12 * f + 4 * n + 4 * t * f + learn + 4 * c * (2 * n + f) + 28 * f + 4 * n
        flops += f * c * (2 * t + 8 + 2 * t + 2 + 14 + 14 + (2 * t if case["learn"] else 0))
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    """A decimation is fixed to the bit (cost order, placement, summation order are specified); feature sums
    are 32-bit sums whose order is not."""
    return "exact" if case["op"] == "decimate" else {"rel": 1e-5}
