"""Rounds by rings against the oracle, to the bit: vertices with as many facets as a short ring, a pair of lanes and a wave's turn have and one more, rings that
grow from round to round, calls that go on by facets in a later round, facets wound both ways round, repeated (two-sided surfaces) and degenerate ones, batches whose meshes
end at different times, equal costs, and the meshes on either side of the rule that takes a call to them."""
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
    """Up to 10 facets of up to 10 vertices a short ring, up to 16 a pair of lanes' row, more a wave's."""
    V, F = wheels(spokes, closed, 11)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    for keep in (0.8, 0.5, 0.1):
        target = max(1, int(len(V) * keep))
        same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target))


@pytest.mark.parametrize("n_rim", [24, 40, 104])
def test_ring_of_two_hubs(pk, oracle, n_rim):
    """A disc around two neighbouring vertices that become one: its ring grows in the second round (24: from short ones to a row; 104: beyond a wave's lanes)."""
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
    """Meshes that end in different rounds, one that takes no part, more than the workgroups keep in LDS; one with a vertex of a hundred facets."""
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


def joined(parts):
    base = np.concatenate([[0], np.cumsum([len(v) for v, _ in parts])])
    return np.concatenate([v for v, _ in parts]).astype(np.float32), np.concatenate([f + np.int32(base[k]) for k, (_, f) in enumerate(parts)]).astype(np.int32)


@pytest.mark.parametrize("closed", [True, False])
@pytest.mark.parametrize("turned", [0.0, 0.4])
@pytest.mark.parametrize("spokes", [(9, 10), (10, 11, 12), (8, 9, 10, 11)])
def test_edge_of_short_rings(pk, oracle, spokes, closed, turned):
    """Ten facets closed are the last short ring, ten open ones name eleven vertices, eleven are a row by their number; words nine and ten of a short ring lie beside its row.
    With facets wound the other way round first corners are met twice, and fewer fit."""
    V, F = wheels(spokes * 5, closed, 17)
    flip = np.random.default_rng(5).random(len(F)) < turned
    F[flip] = F[flip][:, ::-1]
    ctx = pk.Context(len(V), len(F), 1, device=0)
    for place in (pk.PICASSO_PLACE_MEAN, pk.PICASSO_PLACE_INVERSE):
        ctx.set_placement(place, 1e-3)
        for keep in (0.9, 0.5, 0.1):
            target = max(1, int(len(V) * keep))
            same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target, placement=place, rcond_min=1e-3))


@pytest.mark.parametrize("closed", [True, False])
@pytest.mark.parametrize("spokes", [(16, 17, 18), (63, 64, 65, 66), (127, 128, 129, 130), (255, 256, 257), (40,) * 30, (1023, 1100, 1400)])
@pytest.mark.parametrize("side", [5, 150])
def test_long_rings(pk, oracle, spokes, closed, side):
    """Either side of a pair's row, of a wave's turns (64 facets, 128 and 256) and of what one wave takes (1,024 and one for 64 vertices); few vertices beside them, so that the rounds go on by facets, and many, so that they do not."""
    V, F = joined([meshgen.noisy_grid(side, side, seed=3), wheels(spokes, closed, 23)])
    ctx = pk.Context(len(V), len(F), 1, device=0)
    for keep in (0.8, 0.4, 0.1):
        target = max(1, int(len(V) * keep))
        same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target))


@pytest.mark.parametrize("drop", [0, 1])
@pytest.mark.parametrize("spokes,side", [((60,) * 100, 140), ((280,), 140)])
@pytest.mark.parametrize("two_sided", [False, True])
def test_by_facets_in_a_later_round(pk, oracle, spokes, side, two_sided, drop):
    """A mesh of wheels that takes no part beside a lattice that shrinks: from some round on the wheels' rings are many, or the one is long, for the vertices there are, and the
    rounds go on by facets, with the labels that the rounds before have left.  Two-sided, the rings have every other facet left out, the facets have not."""
    lat = meshgen.noisy_grid(side, side, seed=4)
    if two_sided:
        lat = (lat[0], np.concatenate([lat[1][:2000], lat[1], lat[1][:2000, ::-1]]))
    wheel = wheels(spokes, True, 5)
    parts = [lat, wheel, meshgen.noisy_grid(20, 20, seed=9)]
    V, F = joined(parts)
    nv, nf = [len(v) for v, _ in parts], [len(f) for _, f in parts]
    target = [nv[0] // 50, nv[1], nv[2] // 3]
    ctx = pk.Context(len(V), len(F), 3, device=0)
    ctx.set_option(pk.PICASSO_OPT_DROP_DEGENERATED, drop)
    got = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, target)
    ref = oracle.decimate_batch(V, F, nv, nf, target)
    if drop:
        ref = oracle.drop_unreferenced(ref, ref["nv"])
    same(got, ref)
    assert list(got[4]) == list(ref["nv"]) and list(got[5]) == list(ref["nf"])


@pytest.mark.parametrize("drop", [0, 1])
@pytest.mark.parametrize("w,h,beside", [(3, 3, 20), (40, 30, 1300), (90, 90, 9000)])
def test_two_sided_surfaces(pk, oracle, w, h, beside, drop):
    """Lattices whose facets are there from both sides, beside vertices of no facet, which take the call to rounds by rings: twelve facets and six neighbours a vertex."""
    rng = np.random.default_rng(w)
    V, F = meshgen.noisy_grid(w, h, seed=w)
    order = rng.permutation(2 * len(F))
    for facets in (np.concatenate([F, F[:, ::-1]]), np.concatenate([F, F[:, [1, 0, 2]]])[order], np.concatenate([F, F])):
        f = np.ascontiguousarray(facets, dtype=np.int32)
        v = np.concatenate([V, rng.normal(size=(beside, 3))]).astype(np.float32)
        ctx = pk.Context(len(v), len(f), 1, device=0)
        ctx.set_option(pk.PICASSO_OPT_DROP_DEGENERATED, drop)
        for target in (len(v) - len(V) // 4, len(v) - len(V) // 2, beside + 2):
            ref = oracle.decimate(v, f, target)
            same(ctx.picasso_decimate(dev(v), dev(f), target), oracle.drop_unreferenced(ref) if drop else ref)


@pytest.mark.parametrize("n,m", [(40, 85), (3000, 6600), (20000, 40000)])
@pytest.mark.parametrize("beside", [0, 1])
def test_facets_of_any_vertices(pk, oracle, n, m, beside):
    """Most vertices name more neighbours than a short ring has: the first round goes by facets when its rings have been made; beside twice as many vertices of a lattice it does not."""
    rng = np.random.default_rng(n)
    parts = [(rng.normal(size=(n, 3)), rng.integers(0, n, (m, 3)).astype(np.int32))]
    if beside:
        side = int((2 * n) ** 0.5) + 2
        parts.append(meshgen.noisy_grid(side, side, seed=n))
    V, F = joined(parts)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    for keep in (0.8, 0.4, 0.1):
        target = max(1, int(len(V) * keep))
        same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target))


def test_bracketed_kernels_of_every_way(pk):
    """A launch and its bytes for every round, by the way that the round went: by rings, by facets where the first round by rings was given up, by facets from some round on."""
    rng = np.random.default_rng(1)
    lat, wheel = meshgen.noisy_grid(140, 140, seed=4), wheels((60,) * 100, True, 5)
    any_three = (rng.normal(size=(3000, 3)).astype(np.float32), rng.integers(0, 3000, (6600, 3)).astype(np.int32))

    def measured(parts, rounds):
        V, F = joined(parts)
        nv, nf = [len(v) for v, _ in parts], [len(f) for _, f in parts]
        ctx = pk.Context(len(V), len(F), len(parts), device=0)
        ctx.set_option(pk.PICASSO_OPT_KERNEL_TIMING, 1)
        ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, rounds)
        left = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, [max(1, nv[0] // 60)] + nv[1:])[1].shape[0]
        got = [ctx.picasso_kernel_timing(k) for k in (pk.PICASSO_KERNEL_UNIQUE_COST, pk.PICASSO_KERNEL_SUBROUND0)]
        return len(V), len(F), left, [g["launches"] for g in got], [g["bytes_total"] for g in got]

    n, m, _, launches, nbytes = measured([lat], 1)
    assert launches == [1, 1] and nbytes == [152 * n, 16 * n]
    n, m, _, launches, nbytes = measured([any_three], 1)
    assert launches == [1, 1] and nbytes == [24 * m + 72 * n, 24 * m + 32 * n]
    n, before, by_rings = len(lat[0]) + len(wheel[0]), 0, []
    for rounds in range(1, 8):
        _, _, left, launches, nbytes = measured([lat, wheel], rounds)
        assert launches == [rounds, rounds]
        by_rings.append(nbytes[1] - before == 16 * n)
        assert by_rings[-1] or nbytes[1] - before > 32 * n
        n, before = left, nbytes[1]
    assert by_rings[0] and not by_rings[-1] and by_rings == sorted(by_rings, reverse=True)
