"""Rounds by rings against the oracle, to the bit: vertices with as many facets as a short ring, its two lines and a block of rows take and one more, rings
that outgrow their rows in a later round, facets wound both ways round, repeated and degenerate ones, batches whose meshes end at different times, equal costs, and the
meshes on either side of the rule that takes a call to them."""
import numpy as np
import pytest

from paper_2103_15076_amd import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_15076_amd
    return paper_2103_15076_amd


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def same(got, ref):
    st, vo, fo, cid = got[:4]
    assert st == ref["status"]
    np.testing.assert_array_equal(cid.cpu().numpy(), ref["cluster_id"])
    np.testing.assert_array_equal(fo.cpu().numpy(), ref["facets"])
    np.testing.assert_array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))


def wheels(spokes, closed, seed):
    """Wheels of these many spokes in a row, each with a lattice of its own beside it so that vertices have few facets on average."""
    rng = np.random.default_rng(seed)
    V, F, at = [], [], 0
    for k, n in enumerate(spokes):
        a = np.arange(n if closed else n + 1) * 2 * np.pi / (n if closed else n + 1)
        rim = np.stack([np.cos(a), np.sin(a), 0.2 * rng.normal(size=len(a))], 1) + [3 * k, 0, 0]
        V += [[[3 * k, 0, 1.0]], rim]
        i = np.arange(n)
        F.append(np.stack([np.full(n, at), at + 1 + i, at + 1 + (i + 1) % len(a)], 1))
        at += 1 + len(a)
        v, f = meshgen.noisy_grid(6, 5, seed=seed + k)
        V.append(v + np.float32([3 * k, 5, 0]))
        F.append(f + at)
        at += len(v)
    return np.concatenate(V).astype(np.float32), np.concatenate(F).astype(np.int32)


@pytest.mark.parametrize("closed", [True, False])
@pytest.mark.parametrize("spokes", [(3, 4, 5, 6, 7, 8, 9), (8, 9, 15, 16, 17), (16, 17, 31, 33, 63, 64), (65,), (64, 200)])
def test_lengths_of_rings(pk, oracle, spokes, closed):
    """Up to 8 facets a short ring, up to 16 in lines, up to 64 in a block; beyond, the round goes by facets."""
    V, F = wheels(spokes, closed, 11)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    for keep in (0.8, 0.5, 0.1):
        target = max(1, int(len(V) * keep))
        same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target))


@pytest.mark.parametrize("n_rim", [24, 40, 104])
def test_ring_of_two_hubs(pk, oracle, n_rim):
    """A disc around two neighbouring vertices that become one: its ring grows beyond a line, a row and (104) what a row takes at most, so that the second
    round goes by facets, on facets that are still the input's."""
    rng = np.random.default_rng(n_rim)
    a = np.arange(n_rim) * 2 * np.pi / n_rim
    h = n_rim // 2
    V = np.concatenate([[[0.05, 0, 0], [-0.05, 0, 0]], np.stack([np.cos(a - np.pi / 2), np.sin(a - np.pi / 2), 0.3 * rng.normal(size=n_rim)], 1)])
    F = [[0, 2 + i, 2 + i + 1] for i in range(h)] + [[1, 2 + i, 2 + (i + 1) % n_rim] for i in range(h, n_rim)] + [[0, 2 + h, 1], [1, 2, 0]]
    v, f = meshgen.noisy_grid(20, 15, seed=2)
    V, F = np.concatenate([V, v + [5, 0, 0]]).astype(np.float32), np.concatenate([np.int32(F), f + np.int32(len(V))]).astype(np.int32)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, 1)
    _, _, _, cid = ctx.picasso_decimate(dev(V), dev(F), 1)
    assert cid[0] == cid[1], "the hubs are to become one in the first round"
    ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, -1)
    for drop in (0, 1):
        ctx.set_option(pk.PICASSO_OPT_DROP_DEGENERATED, drop)
        for target in (int(0.4 * len(V)), 60, 12, 1):
            ref = oracle.decimate(V, F, target)
            same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.drop_unreferenced(ref) if drop else ref)


@pytest.mark.parametrize("turned,repeated,degenerate", [(0.5, 0.0, 0.0), (0.0, 0.15, 0.0), (0.3, 0.1, 0.1)])
@pytest.mark.parametrize("n", [5, 64, 129, 4000])
def test_turned_repeated_and_degenerate_facets(pk, oracle, n, turned, repeated, degenerate):
    rng = np.random.default_rng(n)
    w = max(3, int(np.sqrt(n)))
    V, F = meshgen.noisy_grid(w, w, seed=n)
    flip, again, flat = (rng.random(len(F)) < p for p in (turned, repeated, degenerate))
    F[flip] = F[flip][:, ::-1]
    F[again] = F[rng.integers(0, len(F), again.sum())]
    F[flat, 2] = F[flat, rng.integers(0, 2, flat.sum())]
    ctx = pk.Context(len(V), len(F), 1, device=0)
    for place in (pk.PICASSO_PLACE_MEAN, pk.PICASSO_PLACE_INVERSE):
        ctx.set_placement(place, 1e-3)
        for keep in (0.7, 0.2):
            target = max(1, int(len(V) * keep))
            same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target, placement=place, rcond_min=1e-3))


@pytest.mark.parametrize("facets_per_vertex", [2.2, 2.3, 4.0])
def test_rule_of_facets(pk, oracle, facets_per_vertex):
    """Either side of the number of facets up to which a call goes by rings: a lattice with more or fewer of its facets there again the other way round."""
    V, F = meshgen.noisy_grid(40, 30, seed=3)
    F = np.concatenate([F, F[:, ::-1]])[:int(len(V) * facets_per_vertex)].astype(np.int32)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    for keep in (0.6, 0.3, 0.05):
        target = max(1, int(len(V) * keep))
        same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target))


@pytest.mark.parametrize("side", [2, 40])
def test_equal_costs(pk, oracle, side):
    V, F = meshgen.noisy_grid(side, side, seed=1)
    V[:, 2] = 0
    ctx = pk.Context(len(V), len(F), 1, device=0)
    for keep in (0.7, 0.25):
        target = max(1, int(len(V) * keep))
        same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target))


@pytest.mark.parametrize("meshes,one_is_wide", [(5, False), (5, True), (70, False)])
def test_batches(pk, oracle, meshes, one_is_wide):
    """Meshes that end in different rounds, one that takes no part, more than the workgroups keep in LDS; one vertex too many facets takes all of them to the other way."""
    parts = [meshgen.noisy_grid(6 + k % 9, 5 + k % 7, seed=k) for k in range(meshes)]
    if one_is_wide:
        parts[3] = wheels((100, 12), True, 3)
    nv, nf = [len(p[0]) for p in parts], [len(p[1]) for p in parts]
    base = np.concatenate([[0], np.cumsum(nv)])
    V, F = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] + np.int32(base[k]) for k, p in enumerate(parts)])
    targets = [n if k == 1 else max(1, int(n * (0.1 + 0.8 * (k % 4) / 3))) for k, n in enumerate(nv)]
    ctx = pk.Context(len(V), len(F), meshes, device=0)
    st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, targets)
    vo, fo, cid = vo.cpu().numpy(), fo.cpu().numpy(), cid.cpu().numpy()
    at_v = at_f = 0
    for k, (v, f) in enumerate(parts):
        ref = oracle.decimate(v, f, targets[k])
        np.testing.assert_array_equal(cid[base[k]:base[k + 1]] - at_v, ref["cluster_id"])
        np.testing.assert_array_equal(vo[at_v:at_v + nvo[k]].view(np.uint32), ref["verts"].view(np.uint32))
        np.testing.assert_array_equal(fo[at_f:at_f + nfo[k]] - at_v, ref["facets"])
        at_v, at_f = at_v + nvo[k], at_f + nfo[k]
