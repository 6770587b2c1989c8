"""GPU parity: the HIP path (through the C-ABI binding) against the CPU oracle,
element by element on the same seeded inputs.

Bar (the benchmark spec): bit-exact cluster_id, facet list and counts; positions within
1e-5 relative (they are expected to be bit-identical as well, and that is
asserted where noted).
"""
import numpy as np
import pytest

from paper_2103_15076_amd import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pk():
    import paper_2103_15076_amd as p
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p.load_library()  # raises if the HIP library has not been built
    return p


@pytest.fixture(scope="module")
def ctx(pk):
    c = pk.Context(1_300_000, 2_500_000, 16, device=0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def ctx16k(pk):
    c = pk.Context(200_000, 400_000, 64, device=0)
    yield c
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def assert_same_result(st, vo, fo, cid, ref, exact_positions=True):
    assert st == ref["status"]
    vo, fo, cid = vo.cpu().numpy(), fo.cpu().numpy(), cid.cpu().numpy()
    assert vo.shape[0] == ref["verts"].shape[0], (vo.shape, ref["verts"].shape)
    assert fo.shape[0] == ref["facets"].shape[0], (fo.shape, ref["facets"].shape)
    assert np.array_equal(cid, ref["cluster_id"])
    assert np.array_equal(fo, ref["facets"])
    tol = 1e-5 * np.maximum(1.0, np.abs(ref["verts"]))
    assert np.all(np.abs(vo - ref["verts"]) <= tol)
    if exact_positions:
        assert np.array_equal(vo.view(np.uint32), ref["verts"].view(np.uint32))


# ----------------------------------------------------------------------------
# primitives
# ----------------------------------------------------------------------------

@pytest.mark.parametrize("n,bits", [(1, 32), (63, 7), (4096, 32), (4097, 13), (70001, 32), (1 << 20, 20)])
def test_radix_sort_pairs_u32_is_stable(ctx, n, bits):
    rng = np.random.default_rng(n)
    keys = rng.integers(0, 1 << bits, size=n, dtype=np.uint64).astype(np.uint32)
    vals = np.arange(n, dtype=np.uint32)
    k, v = dev(keys.view(np.int32)), dev(vals.view(np.int32))
    print(f"sort u32 n={n} bits={bits}", flush=True)
    ctx.picasso_radix_sort(k, v, key_bits=bits)
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(k.cpu().numpy().view(np.uint32), keys[order])
    assert np.array_equal(v.cpu().numpy().view(np.uint32), vals[order])


@pytest.mark.parametrize("n,bits,with_vals", [(5, 34, False), (12289, 34, False), (300000, 42, False),
                                              (100000, 36, True), (2500000, 40, False)])
def test_radix_sort_u64(ctx, n, bits, with_vals):
    rng = np.random.default_rng(n + 1)
    keys = rng.integers(0, 1 << bits, size=n, dtype=np.uint64)
    keys[: n // 3] = keys[n // 3: 2 * (n // 3)][: n // 3]   # duplicates
    k = dev(keys.view(np.int64))
    v = dev(np.arange(n, dtype=np.int32)) if with_vals else None
    print(f"sort u64 n={n} bits={bits}", flush=True)
    ctx.picasso_radix_sort(k, v, key_bits=bits)
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(k.cpu().numpy().view(np.uint64), keys[order])
    if with_vals:
        assert np.array_equal(v.cpu().numpy(), order.astype(np.int32))


def _bucket_cases():
    rng = np.random.default_rng(99)
    # (name, keys, bits): evenly spread, ragged, empty buckets, one bucket far beyond the LDS capacity
    yield "uniform34", rng.integers(0, 1 << 34, size=300001, dtype=np.uint64), 34
    yield "tiny", rng.integers(0, 1 << 20, size=37, dtype=np.uint64), 20
    yield "few_bits", rng.integers(0, 1 << 6, size=5000, dtype=np.uint64), 6
    yield "nine_bits", rng.integers(0, 1 << 9, size=70000, dtype=np.uint64), 9
    k = rng.integers(0, 1 << 32, size=200000, dtype=np.uint64)
    k[:120000] = (np.uint64(5) << np.uint64(24)) | (k[:120000] & np.uint64(0xFFFFFF))   # 120k keys share the top byte
    rng.shuffle(k)
    yield "skewed_oversize", k, 32
    # one bucket of 256 holds 20,000 keys, more than LDS takes, but spread over its 512 groups (about 40 keys
    # each): sorted in parts of whole groups
    k = rng.integers(0, 1 << 34, size=200000, dtype=np.uint64)
    k[:20000] = (np.uint64(5) << np.uint64(26)) | (k[:20000] & np.uint64((1 << 26) - 1))
    rng.shuffle(k)
    yield "oversize_in_parts", k, 34
    k = np.full(30000, (7 << 20) | 12345, np.uint64)   # all equal: one oversize bucket, stability only
    yield "all_equal", k, 28
    yield "full", rng.integers(0, 1 << 40, size=1 << 20, dtype=np.uint64), 40
    yield "large4096", rng.integers(0, 1 << 42, size=3000001, dtype=np.uint64), 42
    k = rng.integers(0, 1 << 30, size=1500000, dtype=np.uint64)
    k[:200000] &= np.uint64((1 << 18) - 1)     # 200k keys in bucket 0 of 4096: far beyond the LDS capacity
    rng.shuffle(k)
    yield "large_skewed", k, 30


@pytest.mark.parametrize("name,keys,bits", list(_bucket_cases()), ids=lambda x: x if isinstance(x, str) else "")
@pytest.mark.parametrize("width", [32, 64])
def test_bucket_sort_is_stable_and_handles_uneven_buckets(ctx, name, keys, bits, width):
    if width == 32 and bits > 32:
        keys, bits = keys & np.uint64(0xFFFFFFFF), 32
    n = keys.shape[0]
    vals = np.arange(n, dtype=np.int32)
    k = dev(keys.astype(np.uint32).view(np.int32)) if width == 32 else dev(keys.view(np.int64))
    v = dev(vals)
    print(f"bucket sort {name} n={n} bits={bits} width={width}", flush=True)
    ctx.picasso_bucket_sort(k, v, key_bits=bits)
    order = np.argsort(keys, kind="stable")
    got = k.cpu().numpy().view(np.uint32 if width == 32 else np.uint64)
    assert np.array_equal(got.astype(np.uint64), keys[order])
    assert np.array_equal(v.cpu().numpy(), order.astype(np.int32))
    # keys only
    k2 = dev(keys.astype(np.uint32).view(np.int32)) if width == 32 else dev(keys.view(np.int64))
    ctx.picasso_bucket_sort(k2, None, key_bits=bits)
    assert np.array_equal(k2.cpu().numpy().view(np.uint32 if width == 32 else np.uint64).astype(np.uint64), keys[order])


# ----------------------------------------------------------------------------
# single steps
# ----------------------------------------------------------------------------

def _small_meshes():
    yield "grid", meshgen.noisy_grid(37, 29, seed=3)
    yield "ico", meshgen.icosphere(4, seed=4)
    yield "room", meshgen.room_scene(11, room=(3.0, 2.0, 1.5), n_boxes=5, spacing=0.05)
    yield "flat", meshgen.flat_grid(33, 18, spacing=0.5)


@pytest.mark.parametrize("name,mesh", list(_small_meshes()), ids=lambda x: x if isinstance(x, str) else "")
def test_vertex_quadrics_bit_exact(ctx, oracle, name, mesh):
    V, F = mesh
    print(f"quadrics {name} N={V.shape[0]} F={F.shape[0]}", flush=True)
    Q = ctx.picasso_vertex_quadrics(dev(V), dev(F)).cpu().numpy()
    ref = oracle.vertex_quadrics(V, F)
    assert np.array_equal(Q.view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("name,mesh", list(_small_meshes()), ids=lambda x: x if isinstance(x, str) else "")
def test_edges_and_costs_bit_exact(ctx, oracle, name, mesh):
    V, F = mesh
    print(f"edges {name}", flush=True)
    E, cost = ctx.picasso_edge_costs(dev(V), dev(F))
    E, cost = E.cpu().numpy(), cost.cpu().numpy()
    Er = oracle.edges(F)
    assert np.array_equal(E, Er)
    cr, _ = oracle.edge_costs(V, oracle.vertex_quadrics(V, F), Er)
    assert np.array_equal(cost.view(np.uint32), cr.view(np.uint32))


@pytest.mark.parametrize("n,f", [(3, 1), (5, 30_000), (129, 70_000), (257, 9_000), (3_000, 400_000)])
def test_quadrics_and_edges_of_facet_soups(ctx, oracle, n, f):
    """Vertices with more facets than a bucket of the sort holds in LDS, with less bits than the sort's digit; unused vertices."""
    rng = np.random.default_rng(n + f)
    V = rng.standard_normal((n, 3)).astype(np.float32)
    F = rng.integers(0, n, size=(f, 3)).astype(np.int32)
    F[F == n // 2] = 0  # ... which is in no facet then
    print(f"soup N={n} F={f}", flush=True)
    Q = ctx.picasso_vertex_quadrics(dev(V), dev(F)).cpu().numpy()
    ref = oracle.vertex_quadrics(V, F)
    assert np.array_equal(Q.view(np.uint32), ref.view(np.uint32))
    E, cost = ctx.picasso_edge_costs(dev(V), dev(F))
    Er = oracle.edges(F)
    assert np.array_equal(E.cpu().numpy(), Er)
    cr, _ = oracle.edge_costs(V, ref, Er)
    assert np.array_equal(cost.cpu().numpy().view(np.uint32), cr.view(np.uint32))


@pytest.mark.parametrize("n,f", [(12, 1), (12, 2), (12, 3), (40, 255), (40, 256), (300, 4_095), (300, 4_096), (9_000, 65_535), (9_000, 65_537)])
def test_repeated_facets_of_any_number(ctx, oracle, n, f):
    """The first of equal facets stays, in whichever order they name the corners; a third have one vertex in common.
    The final facets' table keeps a facet's index in as many bits as their number takes."""
    rng = np.random.default_rng(n + f)
    V = rng.standard_normal((n, 3)).astype(np.float32)
    F = rng.integers(0, n, size=(max(f // 2, 1), 3)).astype(np.int32)
    F[::3, 1] = 0
    again = rng.integers(0, F.shape[0], size=f - F.shape[0])
    F = np.concatenate([F, rng.permuted(F[again], axis=1)])[rng.permutation(f)]
    print(f"repeated N={n} F={f}", flush=True)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), n - max(n // 6, 1))
    assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, n - max(n // 6, 1)))


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, 1_250_000])
def test_few_facets_among_very_many_vertices(ctx, oracle, n):
    """Beyond 2^20 vertices the bits of an edge key below an 8-bit digit do not fit 32 bits."""
    Vg, Fg = meshgen.noisy_grid(50, 40, seed=9)
    at = np.sort(np.random.default_rng(n).choice(n, size=Vg.shape[0], replace=False))
    at[-1] = n - 1
    V = np.zeros((n, 3), np.float32)
    V[at] = Vg
    F = at[Fg].astype(np.int32)
    print(f"sparse N={n}", flush=True)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), n - 1200)
    assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, n - 1200))


# ----------------------------------------------------------------------------
# whole path
# ----------------------------------------------------------------------------

@pytest.mark.parametrize("name,mesh", list(_small_meshes()), ids=lambda x: x if isinstance(x, str) else "")
@pytest.mark.parametrize("frac,max_rounds", [(0.6, -1), (0.26, 1), (0.26, -1), (0.05, -1), (0.0, -1)])
def test_decimate_matches_oracle(pk, ctx, oracle, name, mesh, frac, max_rounds):
    V, F = mesh
    target = max(1, int(V.shape[0] * frac))
    print(f"decimate {name} N={V.shape[0]} target={target} max_rounds={max_rounds}", flush=True)
    ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, max_rounds)
    try:
        st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
    finally:
        ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, -1)
    ref = oracle.decimate(V, F, target, max_rounds=max_rounds)
    if max_rounds >= 0 and ref["verts"].shape[0] > target:
        st = ref["status"]  # a capped run is not a budget warning on either side
    assert_same_result(st, vo, fo, cid, ref)


@pytest.mark.parametrize("block_max,radix_select", [(0, 0), (0, 1), (1 << 15, 1)],
                         ids=["whole_chip", "whole_chip_old_option_on", "one_workgroup_per_mesh"])
def test_budget_step_every_way(pk, ctx, oracle, block_max, radix_select):
    """The last round keeps a mesh's cheapest pairs by histogram passes of the whole chip over its vertices or by a
    search inside one workgroup per mesh (PICASSO_OPT_TRUNC_SELECT is accepted and changes nothing); against the
    oracle, on meshes with distinct costs and with nothing but ties, alone and in a batch (budgets of 1 pair, of
    all but 1 pair, and in between)."""
    ctx.set_option(pk.PICASSO_OPT_TRUNC_BLOCK_MAX, block_max)
    ctx.set_option(pk.PICASSO_OPT_TRUNC_SELECT, radix_select)
    try:
        for name, (V, F) in _small_meshes():
            for frac in (0.9, 0.55):
                target = int(V.shape[0] * frac)
                print(f"budget {name} target={target} block_max={block_max}", flush=True)
                st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
                assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))
        parts = [meshgen.noisy_grid(30, 22, seed=1), meshgen.flat_grid(21, 17, spacing=0.25),
                 meshgen.icosphere(3, seed=2), meshgen.noisy_grid(12, 12, seed=3)]
        nv = [p[0].shape[0] for p in parts]
        nf = [p[1].shape[0] for p in parts]
        off = np.cumsum([0] + nv)
        V = np.concatenate([p[0] for p in parts])
        F = np.concatenate([p[1] + off[i] for i, p in enumerate(parts)]).astype(np.int32)
        for tg in ([nv[0] - 1, nv[1] - 1, nv[2], nv[3] - 1],          # one pair each (one mesh untouched)
                   [nv[0] - 100, nv[1] // 2, nv[2] - 7, nv[3] - 30]):
            print(f"budget batch targets={tg} block_max={block_max}", flush=True)
            st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
            ref = oracle.decimate_batch(V, F, nv, nf, tg)
            assert st == ref["status"]
            assert nvo.tolist() == ref["nv"].tolist() and nfo.tolist() == ref["nf"].tolist()
            assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
            assert np.array_equal(fo.cpu().numpy(), ref["facets"])
            assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))
    finally:
        ctx.set_option(pk.PICASSO_OPT_TRUNC_BLOCK_MAX, 1 << 15)
        ctx.set_option(pk.PICASSO_OPT_TRUNC_SELECT, 1)


@pytest.mark.parametrize("meshes", [7, 8, 9, 65])
@pytest.mark.parametrize("block_max", [0, 40, 150, 1 << 15])
def test_budget_step_of_a_batch_where_meshes_take_different_ways(pk, oracle, meshes, block_max):
    """Meshes of about 10 to 480 pairs: with a limit in between, the short runs go to one workgroup each and the long ones
    to the whole chip (eight meshes at a time), in one call, and each is cut once."""
    kinds = [meshgen.noisy_grid(30, 34, seed=1), meshgen.flat_grid(9, 7, spacing=0.25), meshgen.icosphere(3, seed=2),
             meshgen.flat_grid(25, 20, spacing=0.5), meshgen.noisy_grid(12, 12, seed=3), meshgen.icosphere(1, seed=5),
             meshgen.noisy_grid(6, 9, seed=4), meshgen.flat_grid(18, 17, spacing=0.25)]
    parts = [kinds[b % 8] for b in range(meshes)]
    nv, nf = [p[0].shape[0] for p in parts], [p[1].shape[0] for p in parts]
    off = np.cumsum([0] + nv)
    V = np.concatenate([p[0] for p in parts])
    F = np.concatenate([p[1] + off[i] for i, p in enumerate(parts)]).astype(np.int32)
    ctx = pk.Context(V.shape[0], F.shape[0], meshes, device=0)
    try:
        ctx.set_option(pk.PICASSO_OPT_TRUNC_BLOCK_MAX, block_max)
        for keep in (0.95, 0.7, 0.3):
            tg = [int(n * keep) for n in nv]
            print(f"budget of {meshes} meshes keep={keep} block_max={block_max}", flush=True)
            st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
            ref = oracle.decimate_batch(V, F, nv, nf, tg)
            assert st == ref["status"]
            assert nvo.tolist() == ref["nv"].tolist() == tg and nfo.tolist() == ref["nf"].tolist()
            assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
            assert np.array_equal(fo.cpu().numpy(), ref["facets"])
            assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))
    finally:
        ctx.close()


def test_histogram_passes_of_the_budget_step_on_clustered_and_tied_cost_keys(pk, ctx, oracle):
    """A single mesh whose last round forms more pairs than the per-mesh search is allowed here: the
    cost key at the budget is found digit by digit.  Flat lattices (every cost key equal: the budget cuts
    through one run of ties, in edge order), a lattice with a few creases (two key values), noisy
    surfaces (keys spread over many leading digits) and the room (keys clustered in a few exponents),
    each at budgets of 1 pair, about half the pairs, and all but 1."""
    ctx.set_option(pk.PICASSO_OPT_TRUNC_BLOCK_MAX, 0)
    try:
        crease_v, crease_f = meshgen.flat_grid(40, 30, spacing=0.5)
        crease_v = crease_v.copy()
        crease_v[::7, 2] += 0.25
        room_v, room_f = meshgen.room_scene(seed=77, n_boxes=6, spacing=0.25)
        for name, (V, F) in (("flat", meshgen.flat_grid(64, 48, spacing=0.25)), ("creases", (crease_v, crease_f)),
                             ("noisy", meshgen.noisy_grid(80, 70, seed=9)), ("sphere", meshgen.icosphere(5, seed=4)),
                             ("room", (room_v, room_f))):
            N = V.shape[0]
            one_round = oracle.decimate(V, F, 1, max_rounds=1)
            pairs = N - one_round["verts"].shape[0]       # pairs the first round would form without a budget
            for remove in (1, pairs // 2, pairs - 1):
                target = N - remove
                print(f"histogram passes {name} N={N} pairs={pairs} target={target}", flush=True)
                st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
                assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))
    finally:
        ctx.set_option(pk.PICASSO_OPT_TRUNC_BLOCK_MAX, 1 << 15)


def test_adversarial_small_meshes(ctx, oracle):
    rng = np.random.default_rng(5)
    cases = {}
    # random facet soup: non-manifold, duplicate facets, repeated indices, isolated vertices
    V = rng.normal(size=(60, 3)).astype(np.float32)
    F = rng.integers(0, 50, size=(150, 3)).astype(np.int32)
    F[10] = F[3]
    F[11] = F[3][::-1]
    F[12] = [7, 7, 9]
    cases["soup"] = (V, F, 9)
    # one triangle and isolated vertices: the budget cannot be met
    cases["stuck"] = (rng.normal(size=(8, 3)).astype(np.float32), np.array([[0, 1, 2]], np.int32), 2)
    # no facets at all
    cases["nofacets"] = (rng.normal(size=(5, 3)).astype(np.float32), np.zeros((0, 3), np.int32), 2)
    # exact ties everywhere (flat lattice): order decided by the edge index alone
    Vf, Ff = meshgen.flat_grid(40, 25)
    cases["ties"] = (Vf, Ff, 100)
    # two vertices
    cases["pair"] = (np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0]], np.float32), np.array([[0, 1, 2]], np.int32), 1)
    for name, (V, F, target) in cases.items():
        print(f"adversarial {name}", flush=True)
        st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
        assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))


def test_hub_vertices_and_uneven_buckets_in_the_pipeline(ctx, oracle):
    """Meshes whose keys are NOT evenly spread: a fan around one hub vertex (its incidences and
    edges all fall into one sort bucket, far more than LDS holds) and a mesh whose vertex count
    is just above a power of two (half of the id range empty)."""
    rng = np.random.default_rng(21)
    # fan: hub 0 joined to a ring of 30000 vertices, plus a noisy grid glued on
    n = 30000
    ang = np.linspace(0, 2 * np.pi, n, endpoint=False)
    ring = np.stack([np.cos(ang), np.sin(ang), 0.05 * rng.normal(size=n)], 1)
    V = np.concatenate([[[0, 0, 0.3]], ring]).astype(np.float32)
    F = np.stack([np.zeros(n, np.int64), 1 + np.arange(n), 1 + (np.arange(n) + 1) % n], 1).astype(np.int32)
    Vg, Fg = meshgen.noisy_grid(40, 40, seed=6)
    V2 = np.concatenate([V, Vg + np.float32([3, 0, 0])]).astype(np.float32)
    F2 = np.concatenate([F, Fg + V.shape[0]]).astype(np.int32)
    for target in (V2.shape[0] // 2, V2.shape[0] // 7):
        print(f"hub fan N={V2.shape[0]} target={target}", flush=True)
        st, vo, fo, cid = ctx.picasso_decimate(dev(V2), dev(F2), target)
        assert_same_result(st, vo, fo, cid, oracle.decimate(V2, F2, target))
    # hub as the LAST vertex (it is the larger end of every edge)
    perm = np.arange(V.shape[0])[::-1].copy()
    inv = np.empty_like(perm)
    inv[perm] = np.arange(perm.size)
    V3, F3 = V[perm], inv[F].astype(np.int32)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V3), dev(F3), 5000)
    assert_same_result(st, vo, fo, cid, oracle.decimate(V3, F3, 5000))
    # vertex count just above a power of two
    Vp, Fp = meshgen.noisy_grid(257, 256, seed=8)     # 65792 = 2^16 + 256
    st, vo, fo, cid = ctx.picasso_decimate(dev(Vp), dev(Fp), 20000)
    assert_same_result(st, vo, fo, cid, oracle.decimate(Vp, Fp, 20000))


def test_batch_of_many_small_meshes(ctx16k, oracle):
    """64 meshes of different kinds and sizes in one call, budgets from 'nothing to do' to 'to one vertex'."""
    rng = np.random.default_rng(33)
    parts, tg = [], []
    for b in range(64):
        kind = b % 4
        if kind == 0:
            p = meshgen.noisy_grid(int(rng.integers(3, 30)), int(rng.integers(3, 30)), seed=100 + b)
        elif kind == 1:
            p = meshgen.icosphere(int(rng.integers(0, 4)), seed=100 + b)
        elif kind == 2:
            p = meshgen.flat_grid(int(rng.integers(2, 20)), int(rng.integers(2, 20)))
        else:
            p = meshgen.room_scene(100 + b, room=(1.0, 1.0, 0.5), n_boxes=1, spacing=0.1)
        parts.append(p)
        n = p[0].shape[0]
        tg.append(int(max(1, [n, n - 1, n // 2, n // 5, 1][b % 5])))
    nv = [p[0].shape[0] for p in parts]
    nf = [p[1].shape[0] for p in parts]
    off = np.cumsum([0] + nv)
    V = np.concatenate([p[0] for p in parts])
    F = np.concatenate([p[1] + off[i] for i, p in enumerate(parts)]).astype(np.int32)
    st, vo, fo, cid, nvo, nfo = ctx16k.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
    ref = oracle.decimate_batch(V, F, nv, nf, tg)
    assert st == ref["status"]
    assert nvo.tolist() == ref["nv"].tolist() and nfo.tolist() == ref["nf"].tolist()
    assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
    assert np.array_equal(fo.cpu().numpy(), ref["facets"])
    assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))


def test_zero_rounds_copies_input(ctx):
    V, F = meshgen.noisy_grid(9, 9, seed=1)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), 81)
    assert st == 0 and np.array_equal(vo.cpu().numpy(), V) and np.array_equal(fo.cpu().numpy(), F)
    assert np.array_equal(cid.cpu().numpy(), np.arange(81))


def test_error_codes_and_untouched_outputs(pk, ctx):
    V, F = meshgen.noisy_grid(20, 20, seed=1)
    vo = torch.full((400, 3), 7.0, device="cuda:0")
    fo = torch.full((F.shape[0], 3), 7, dtype=torch.int32, device="cuda:0")
    cid = torch.full((400,), 7, dtype=torch.int32, device="cuda:0")
    Fb = F.copy()
    Fb[17, 2] = 400
    st, *_ = ctx.picasso_decimate(dev(V), dev(Fb), 100, vo, fo, cid, check=False)
    assert st == pk.PICASSO_ERR_BAD_INDEX
    Fb[17, 2] = -3
    st, *_ = ctx.picasso_decimate(dev(V), dev(Fb), 100, vo, fo, cid, check=False)
    assert st == pk.PICASSO_ERR_BAD_INDEX
    Vb = V.copy()
    Vb[33, 1] = np.inf
    st, *_ = ctx.picasso_decimate(dev(Vb), dev(F), 100, vo, fo, cid, check=False)
    assert st == pk.PICASSO_ERR_NONFINITE
    st, *_ = ctx.picasso_decimate(dev(Vb), dev(F), 400, vo, fo, cid, check=False)   # zero rounds still validates
    assert st == pk.PICASSO_ERR_NONFINITE
    st, *_ = ctx.picasso_decimate(dev(V), dev(F), 0, vo, fo, cid, check=False)
    assert st == pk.PICASSO_ERR_INVALID_ARG
    assert torch.all(vo == 7.0) and torch.all(fo == 7) and torch.all(cid == 7)
    small = pk.Context(100, 100, 1)
    st, *_ = small.picasso_decimate(dev(V), dev(F), 100, check=False)
    assert st == pk.PICASSO_ERR_WORKSPACE
    small.close()
    # the context is still usable after errors
    st, vo2, fo2, cid2 = ctx.picasso_decimate(dev(V), dev(F), 100)
    assert st == 0 and vo2.shape[0] == 100


def test_run_to_run_determinism(ctx):
    V, F = meshgen.room_scene(3, room=(4.0, 3.0, 2.0), n_boxes=6, spacing=0.04)
    a = None
    for rep in range(5):
        st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), V.shape[0] // 5)
        b = (vo.cpu().numpy().tobytes(), fo.cpu().numpy().tobytes(), cid.cpu().numpy().tobytes())
        if a is None:
            a = b
        assert a == b, f"run {rep} differs"


def test_batch_matches_oracle_and_independent_runs(ctx, oracle):
    parts = [meshgen.noisy_grid(30, 22, seed=1), meshgen.icosphere(3, seed=2), meshgen.noisy_grid(12, 12, seed=3),
             meshgen.room_scene(8, room=(2.0, 2.0, 1.0), n_boxes=3, spacing=0.06)]
    nv = [p[0].shape[0] for p in parts]
    nf = [p[1].shape[0] for p in parts]
    tg = [100, 642, 7, nv[3] // 9]    # the sphere needs zero rounds; others 1..4 rounds
    off = np.cumsum([0] + nv)
    V = np.concatenate([p[0] for p in parts])
    F = np.concatenate([p[1] + off[i] for i, p in enumerate(parts)]).astype(np.int32)
    print("batch of 4", flush=True)
    st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
    ref = oracle.decimate_batch(V, F, nv, nf, tg)
    assert st == ref["status"]
    assert nvo.tolist() == ref["nv"].tolist() and nfo.tolist() == ref["nf"].tolist()
    assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
    assert np.array_equal(fo.cpu().numpy(), ref["facets"])
    assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))


# ----------------------------------------------------------------------------
# the benchmark configurations at full size
# ----------------------------------------------------------------------------

@pytest.mark.parametrize("name", ["grid64", "icosphere6", "room115k", "scene1p2m"])
def test_config_full_size(ctx, oracle, name):
    c = meshgen.config(name)
    V, F, target = c["verts"], c["facets"], int(c["target"][0])
    print(f"config {name}: N={V.shape[0]} F={F.shape[0]} target={target}", flush=True)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
    print("  gpu done; oracle...", flush=True)
    ref = oracle.decimate(V, F, target)
    assert_same_result(st, vo, fo, cid, ref)
    assert vo.shape[0] == target


def test_single_stream_and_two_stream_first_round_agree(pk, ctx):
    """The first round's edge sort shares its launches with the sort for the vertex quadrics, or (option off) follows
    it; both schedules must give the same bytes, call after call."""
    c = meshgen.config("scene1p2m")
    V, F, target = dev(c["verts"]), dev(c["facets"]), int(c["target"][0])
    res = []
    try:
        for overlap in (1, 0, 1, 1):
            ctx.set_option(pk.PICASSO_OPT_OVERLAP, overlap)
            print(f"overlap={overlap}", flush=True)
            st, vo, fo, cid = ctx.picasso_decimate(V, F, target)
            torch.cuda.synchronize()
            res.append((st, vo.cpu().numpy().tobytes(), fo.cpu().numpy().tobytes(), cid.cpu().numpy().tobytes()))
    finally:
        ctx.set_option(pk.PICASSO_OPT_OVERLAP, 1)
    assert all(r == res[0] for r in res[1:])


def test_room115k_with_scrambled_numbering(ctx, oracle):
    """The headline mesh with vertex ids and facet order permuted at random (the 256-bucket sorts with
    no locality in their keys)."""
    c = meshgen.config("room115k")
    V, F, target = c["verts"], c["facets"], int(c["target"][0])
    rng = np.random.default_rng(321)
    perm = rng.permutation(V.shape[0])
    V2 = np.empty_like(V)
    V2[perm] = V
    F2 = perm[F].astype(np.int32)[rng.permutation(F.shape[0])]
    print(f"scrambled room115k: N={V2.shape[0]} F={F2.shape[0]} target={target}", flush=True)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V2), dev(F2), target)
    assert_same_result(st, vo, fo, cid, oracle.decimate(V2, F2, target))


def test_large_mesh_with_scrambled_numbering(ctx, oracle):
    """Vertex ids and facet order of a 400k-vertex scene are permuted at random, so neighbouring corners
    of the facet array share no leading index bits: the sorts lose the locality their fast paths use
    (waves whose keys fall into one bucket) and must give the same mesh all the same."""
    V, F, _ = meshgen.room_scene_sized(77, 400_000)
    rng = np.random.default_rng(123)
    perm = rng.permutation(V.shape[0])          # new id of old vertex i
    V2 = np.empty_like(V)
    V2[perm] = V
    F2 = perm[F].astype(np.int32)[rng.permutation(F.shape[0])]
    target = V.shape[0] // 3
    print(f"scrambled: N={V2.shape[0]} F={F2.shape[0]} target={target}", flush=True)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V2), dev(F2), target)
    print("  gpu done; oracle...", flush=True)
    assert_same_result(st, vo, fo, cid, oracle.decimate(V2, F2, target))


def test_batch_of_more_meshes_than_the_tail_tallies_in_lds(pk, oracle):
    """1,100 tiny meshes in one call: above 1,024 meshes the selection tail counts pairs through
    memory instead of LDS; budgets bind in many meshes at once (one budget workgroup per mesh)."""
    rng = np.random.default_rng(9)
    parts = []
    for k in range(1100):
        nx, ny = int(rng.integers(3, 7)), int(rng.integers(3, 7))
        parts.append(meshgen.noisy_grid(nx, ny, seed=1000 + k))
    nv = [p[0].shape[0] for p in parts]
    nf = [p[1].shape[0] for p in parts]
    off = np.cumsum([0] + nv)
    V = np.concatenate([p[0] for p in parts])
    F = np.concatenate([p[1] + off[i] for i, p in enumerate(parts)]).astype(np.int32)
    tg = [max(2, int(n * f)) for n, f in zip(nv, rng.uniform(0.3, 1.0, size=len(nv)))]
    c = pk.Context(V.shape[0], F.shape[0], len(parts), device=0)
    try:
        print(f"batch of {len(parts)}: N={V.shape[0]} F={F.shape[0]}", flush=True)
        st, vo, fo, cid, nvo, nfo = c.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
        ref = oracle.decimate_batch(V, F, nv, nf, tg)
        assert st == ref["status"]
        assert nvo.tolist() == ref["nv"].tolist() and nfo.tolist() == ref["nf"].tolist()
        assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
        assert np.array_equal(fo.cpu().numpy(), ref["facets"])
        assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))
    finally:
        c.close()


@pytest.mark.parametrize("what", ["two_sided", "soup", "loose_triangles"])
@pytest.mark.parametrize("seed", [0, 77])
def test_rounds_with_other_than_six_half_edges_per_vertex(ctx, pk, oracle, what, seed):
    """The digit of a later round's edge sort goes by the half-edges to expect of it: twelve per vertex, a hundred and more, and
    none at all (every facet of the first round collapses, and a patch beside them is left)."""
    if what == "two_sided":
        V, F = meshgen.noisy_grid(330, 300, seed=2)
        F = np.stack([F, F[:, ::-1]], 1).reshape(-1, 3)
    elif what == "soup":
        rng = np.random.default_rng(3)
        n, m = 9000, 400_000
        V, a = rng.normal(size=(n, 3)), rng.integers(0, n, m)
        F = np.stack([a, (a + rng.integers(1, 40, m)) % n, (a + rng.integers(41, 80, m)) % n], 1)
    else:
        P, Q = meshgen.noisy_grid(20, 20, seed=4)
        V = np.concatenate([np.random.default_rng(5).normal(size=(360_000, 3)), P])
        F = np.concatenate([np.arange(360_000).reshape(-1, 3), Q + 360_000])
    V, F = V.astype(np.float32), np.ascontiguousarray(F.astype(np.int32))
    target = V.shape[0] // 4
    ctx.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, seed)
    try:
        print(f"{what}: N={V.shape[0]} F={F.shape[0]} target={target} seed={seed}", flush=True)
        st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
    finally:
        ctx.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, 0)
    assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target, shuffle_seed=seed))


def _unwelded_quads(n):
    """n flat squares of two triangles and four vertices of their own."""
    x, y = 2.0 * (np.arange(n) % 50), 2.0 * (np.arange(n) // 50)
    V = np.zeros((n, 4, 3), np.float32)
    for i, (a, b) in enumerate(((0, 0), (1, 0), (0, 1), (1, 1))):
        V[:, i, 0], V[:, i, 1] = x + a, y + b
    F = np.array([[0, 1, 2], [1, 3, 2]]) + 4 * np.arange(n)[:, None, None]
    return V.reshape(-1, 3), F.reshape(-1, 3).astype(np.int32)


@pytest.mark.parametrize("quads", [(950, 950), (1250, 1249, 1), (1792, 1792), (1793, 1792)])
@pytest.mark.parametrize("keep", [0.5, 0.7])
def test_tail_in_which_every_edge_becomes_a_pair(pk, oracle, quads, keep):
    """The first sub-round pairs two corners of every square and leaves the edge between the others, alone: the tail of a batch
    forms as many pairs as it takes edges, up to 3,584 (one more goes back to the host)."""
    parts = [_unwelded_quads(n) for n in quads]
    nv, nf = [p[0].shape[0] for p in parts], [p[1].shape[0] for p in parts]
    base = np.concatenate([[0], np.cumsum(nv)])
    V, F = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] + np.int32(b) for p, b in zip(parts, base)])
    tg = [max(1, int(n * keep)) for n in nv]
    c = pk.Context(V.shape[0], F.shape[0], len(parts), device=0)
    try:
        c.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, 1)
        print(f"squares {quads} targets={tg}", flush=True)
        st, vo, fo, cid, nvo, nfo = c.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
    finally:
        c.close()
    ref = oracle.decimate_batch(V, F, nv, nf, tg)
    assert st == ref["status"]
    assert nvo.tolist() == ref["nv"].tolist() and nfo.tolist() == ref["nf"].tolist()
    assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
    assert np.array_equal(fo.cpu().numpy(), ref["facets"])
    assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))


def test_beyond_the_bucket_sorts(pk, oracle):
    """2.85 M facets = 8.5 M half-edges, more than are partitioned on 12 bits (2^23 keys): the first round's
    incidence and edge keys are partitioned on a wider digit, whose counts lie in memory; the later rounds drop
    back to 12 bits.  Own context (the shared one is smaller)."""
    V, F, _ = meshgen.room_scene_sized(31, 1_500_000, room=(30.0, 20.0, 3.0), n_boxes=300)
    assert 3 * F.shape[0] > (1 << 23)
    target = V.shape[0] // 2
    c = pk.Context(V.shape[0], F.shape[0], 1, device=0)
    try:
        print(f"huge: N={V.shape[0]} F={F.shape[0]} target={target}", flush=True)
        st, vo, fo, cid = c.picasso_decimate(dev(V), dev(F), target)
        print("  gpu done; oracle...", flush=True)
        assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))
    finally:
        c.close()


def test_smaller_meshes_behind_one_with_a_run_of_vertices_without_facets(pk, oracle):
    """A cropped scan that keeps its vertices: the digits of the run (11 bits, 256 vertices each) are empty in its first round's
    sorts, and hold keys in those of the meshes (9 and 10 bits) that follow on the context, and of its own later rounds."""
    V, F = meshgen.noisy_grid(600, 500, seed=5)
    F = F[~((F >= 50_000) & (F < 100_000)).any(1)]
    assert 3 * F.shape[0] > 1 << 20
    c = pk.Context(V.shape[0], F.shape[0], 1, device=0)
    try:
        for w, h in ((400, 300), (500, 300)):
            for name, (Vi, Fi), target in (("cropped", (V, F), 100_000), ("smaller", meshgen.noisy_grid(w, h, seed=w), w * h // 3)):
                print(f"{name}: N={Vi.shape[0]} F={Fi.shape[0]} target={target}", flush=True)
                st, vo, fo, cid = c.picasso_decimate(dev(Vi), dev(Fi), target)
                assert_same_result(st, vo, fo, cid, oracle.decimate(Vi, Fi, target))
    finally:
        c.close()


@pytest.mark.parametrize("what", ["scrambled", "few_vertices"])
def test_very_large_sorts_without_locality(pk, oracle, what):
    """More than 2^23 half-edges where a tile of keys holds as many leading digits as keys (random vertex numbers and
    facet order: digits that find no place in the tile's table), and on so few vertices that the keys would have no
    more bits than the digit (they are made wider)."""
    rng = np.random.default_rng(5)
    if what == "scrambled":
        V, F, _ = meshgen.room_scene_sized(31, 1_500_000, room=(30.0, 20.0, 3.0), n_boxes=300)
        perm = rng.permutation(V.shape[0])
        V2 = np.empty_like(V)
        V2[perm] = V
        V, F = V2, perm[F].astype(np.int32)[rng.permutation(F.shape[0])]
    else:
        V = rng.normal(size=(60, 3)).astype(np.float32)
        F = rng.integers(0, 60, size=(2_900_000, 3)).astype(np.int32)
    assert 3 * F.shape[0] > (1 << 23)
    target = V.shape[0] // 2
    c = pk.Context(V.shape[0], F.shape[0], 1, device=0)
    try:
        print(f"{what}: N={V.shape[0]} F={F.shape[0]} target={target}", flush=True)
        st, vo, fo, cid = c.picasso_decimate(dev(V), dev(F), target)
        print("  gpu done; oracle...", flush=True)
        assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))
    finally:
        c.close()


def test_config_batch_hierarchy(ctx, oracle):
    """16 room meshes through 4 successive levels, each to 40 % of the vertices;
    the cluster maps of all levels are kept and compared."""
    c = meshgen.config("batch16x60k")
    V, F, nv, nf = c["verts"], c["facets"], c["nv"], c["nf"]
    dV, dF = dev(V), dev(F)
    for level in range(c["levels"]):
        tg = (nv.astype(np.int64) * 4 // 10).astype(np.int32)
        print(f"hierarchy level {level}: N={int(nv.sum())} F={int(nf.sum())}", flush=True)
        st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dV, dF, nv, nf, tg)
        ref = oracle.decimate_batch(V, F, nv, nf, tg)
        assert st == ref["status"]
        assert nvo.tolist() == ref["nv"].tolist() == tg.tolist() and nfo.tolist() == ref["nf"].tolist()
        assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
        assert np.array_equal(fo.cpu().numpy(), ref["facets"])
        assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))
        V, F, nv, nf = ref["verts"], ref["facets"], ref["nv"], ref["nf"]
        dV, dF = vo.clone(), fo.clone()


def test_contexts_can_be_created_and_destroyed_many_times(pk):
    """Every context owns device memory, pinned memory, a stream and events: 300 create / use /
    destroy cycles must leave the device's free memory where it was."""
    V, F = meshgen.noisy_grid(12, 12, seed=1)
    dV, dF = dev(V), dev(F)
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    for i in range(300):
        c = pk.Context(50_000, 100_000, 4, device=0)
        if i % 50 == 0:
            st, vo, fo, cid = c.picasso_decimate(dV, dF, 40)
            assert st == 0 and vo.shape[0] == 40
        c.close()
    torch.cuda.synchronize()
    free1, _ = torch.cuda.mem_get_info()
    assert free0 - free1 < 64 << 20, (free0, free1)


def test_on_a_stream_of_the_callers(pk, ctx, oracle):
    """The calls run on the stream they are given: inputs produced on a side stream just before the
    call are seen, outputs are complete when the call returns (it waits for that stream), and work
    queued on the same stream afterwards sees them."""
    V, F = meshgen.icosphere(4, seed=7, jitter=0.05)
    target = V.shape[0] // 4
    ref = oracle.decimate(V, F, target)
    side = torch.cuda.Stream()
    hV, hF = torch.from_numpy(V).pin_memory(), torch.from_numpy(F).pin_memory()
    with torch.cuda.stream(side):
        dV = hV.to("cuda:0", non_blocking=True)
        dF = hF.to("cuda:0", non_blocking=True)
        st, vo, fo, cid = ctx.picasso_decimate(dV, dF, target, stream=side)
        doubled = vo * 2.0
    assert_same_result(st, vo, fo, cid, ref)
    side.synchronize()
    assert np.array_equal(doubled.cpu().numpy(), ref["verts"] * np.float32(2.0))
    # larger input
    c = meshgen.config("scene1p2m")
    V2, F2, t2 = c["verts"], c["facets"], int(c["target"][0])
    with torch.cuda.stream(side):
        d2, f2 = dev(V2), dev(F2)
        st, vo, fo, cid = ctx.picasso_decimate(d2, f2, t2, stream=side)
    assert_same_result(st, vo, fo, cid, oracle.decimate(V2, F2, t2))


@pytest.mark.parametrize("w,h,what", [
    (105, 106, "just below 2^16 half-edges: 8-bit digits"),
    (106, 106, "just above 2^16 half-edges: 9-bit digits"),
    (363, 362, "just below 3 x 2^18 half-edges: 9-bit digits"),
    (364, 363, "just above 3 x 2^18 half-edges: 10-bit digits"),
    (419, 419, "just below 2^20 half-edges: 10-bit digits, one lane per edge in every sub-round"),
    (420, 419, "just above 2^20 half-edges: 11-bit digits, listed sub-rounds"),
    (837, 837, "just below 2^22 half-edges: 11-bit digits"),
    (838, 837, "just above 2^22 half-edges: 12-bit digits"),
])
def test_sizes_on_either_side_of_the_path_switches(ctx, oracle, w, h, what):
    V, F = meshgen.noisy_grid(w, h, seed=w + h, noise=0.004)
    target = V.shape[0] // 3
    print(f"switch {w}x{h}: N={V.shape[0]} F={F.shape[0]} 3F={3 * F.shape[0]} ({what})", flush=True)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
    assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))


@pytest.mark.parametrize("w,keys_per_lane", [(64, 4), (120, 8), (168, 16), (240, 32)])
def test_every_width_of_the_per_mesh_budget_search(ctx, oracle, w, keys_per_lane):
    """One run that forms about 0.45 N pairs and may keep a few hundred, or all but a few, with up to 4, 8, 16 and 32 x 1024
    pairs: one instance of the search releases them itself (up to 4,096), the other leaves it to a kernel of its own."""
    V, F = meshgen.noisy_grid(w, w, seed=w, noise=0.01)
    N = V.shape[0]
    E = oracle.edges(F)
    _, key = oracle.edge_costs(V, oracle.vertex_quadrics(V, F), E)
    _, pairs = oracle.select(E, key, N, N)
    assert (keys_per_lane // 2) * 1024 < pairs <= keys_per_lane * 1024 or keys_per_lane == 4, pairs
    for keep in (300, pairs - 7):
        print(f"budget search w={w}: {pairs} pairs formed, {keep} kept", flush=True)
        st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), N - keep)
        assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, N - keep))
        assert vo.shape[0] == N - keep


@pytest.mark.parametrize("flat", ["all", "half", "none"])
@pytest.mark.parametrize("seed,absorb", [(0, 0), (91, 0), (0, 1), (91, 1)])
def test_per_mesh_budget_search_of_more_keys_than_it_lists(pk, ctx, oracle, flat, seed, absorb):
    """28 k pairs where 16 k are listed: a sample of the costs tells which, unless they are all equal, or half of them are and lie together."""
    V, F = meshgen.noisy_grid(251, 249, seed=6)
    V = V.copy()
    if flat == "all":
        V[:, 2] = 0
    elif flat == "half":
        V[: V.shape[0] // 2, 2] = 0
    ctx.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, seed)
    ctx.set_option(pk.PICASSO_OPT_ABSORB, absorb)
    try:
        n = V.shape[0]
        for remove in (1, n // 5, n // 3, n * 45 // 100 if absorb else n * 2 // 5):
            print(f"search flat={flat} seed={seed} absorb={absorb} remove={remove}", flush=True)
            st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), n - remove)
            assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, n - remove, shuffle_seed=seed, absorb=bool(absorb)))
    finally:
        ctx.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, 0)
        ctx.set_option(pk.PICASSO_OPT_ABSORB, 0)


@pytest.mark.parametrize("batch", [1, 2])
def test_few_sub_rounds_between_looks_of_the_host(pk, ctx, oracle, batch):
    """With only one or two grid-wide sub-rounds per batch the single-workgroup tail finds more live
    edges than it can take, hands back, and the host queues further batches: same result."""
    ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, batch)
    try:
        for name, (V, F) in list(_small_meshes()) + [("room115k", (meshgen.config("room115k")["verts"],
                                                                 meshgen.config("room115k")["facets"]))]:
            target = V.shape[0] // 3
            print(f"sub-round batch {batch}: {name}", flush=True)
            st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
            assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))
    finally:
        ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, 16)


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("seed", [0, 77])
@pytest.mark.parametrize("batch", [1, 3, 16])
def test_listed_sub_rounds(pk, ctx, oracle, flat, seed, batch):
    """Rounds of more than 2^20 half-edges list their live edges from sub-round to sub-round: many of them (every cost equal), one or three
    to a look of the host, with the seeded order; parts of the list that end within a tile."""
    V, F = meshgen.noisy_grid(601, 397, seed=3)
    if flat:
        V = V.copy()
        V[:, 2] = 0
    ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, batch)
    ctx.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, seed)
    try:
        for target in (V.shape[0] * 7 // 10, V.shape[0] // 3):
            print(f"listed flat={flat} seed={seed} batch={batch} target={target}", flush=True)
            st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
            assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target, shuffle_seed=seed))
    finally:
        ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, 16)
        ctx.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, 0)


def test_listed_sub_rounds_of_a_batch_with_meshes_that_rest(ctx, oracle):
    """The edges of meshes that take no part stay out of the lists from the start."""
    parts = [meshgen.noisy_grid(w, h, seed=w) for w, h in ((300, 200), (7, 9), (411, 300), (2, 2), (350, 250))]
    nv, nf = [p[0].shape[0] for p in parts], [p[1].shape[0] for p in parts]
    base = np.concatenate([[0], np.cumsum(nv)])
    V, F = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] + np.int32(b) for p, b in zip(parts, base)])
    target = [nv[0] // 2, nv[1], nv[2], 1, nv[4] // 5]
    print("listed batch", flush=True)
    st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, target)
    ref = oracle.decimate_batch(V, F, nv, nf, target)
    assert list(nvo) == list(ref["nv"]) and list(nfo) == list(ref["nf"])
    assert_same_result(st, vo, fo, cid, ref)


@pytest.mark.parametrize("w,h", [(511, 512), (514, 515), (2_055, 2_053)])
def test_facets_of_a_batch_go_out_from_lists(pk, oracle, w, h):
    """Final facets are listed in segments of 64 to 256, by their number; meshes start within segments, some have no facets left."""
    parts = [meshgen.noisy_grid(a, b, seed=a) for a, b in ((5, 4), (30, 41), (w, h), (2, 2), (3, 2), (71, 50), (2, 3))]
    nv, nf = [p[0].shape[0] for p in parts], [p[1].shape[0] for p in parts]
    base = np.concatenate([[0], np.cumsum(nv)])
    V, F = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] + np.int32(b) for p, b in zip(parts, base)])
    target = [2, nv[1] // 3, nv[2], 1, 2, nv[5] // 2, nv[6]]  # the large one rests
    if w < 1000:
        target[2] = nv[2] // 2
    print(f"lists {sum(nf)}", flush=True)
    ctx = pk.Context(V.shape[0], F.shape[0], len(parts), device=0)
    try:
        st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, target)
    finally:
        ctx.close()
    ref = oracle.decimate_batch(V, F, nv, nf, target)
    assert list(nvo) == list(ref["nv"]) and list(nfo) == list(ref["nf"])
    assert_same_result(st, vo, fo, cid, ref)


@pytest.mark.parametrize("sizes", [[(16, 16)], [(2, 129)], [(127, 129)], [(128, 128)], [(5, 3277)],
                                   [(100, 81), (3, 3), (16, 16), (7, 1143), (2, 2)], [(100, 81), (3, 3), (16, 16), (7, 1145), (2, 2)]])
def test_contraction_that_counts_for_itself(pk, ctx, oracle, sizes):
    """Up to 16,384 vertices (of a round) no count pass runs in front of the contraction."""
    parts = [meshgen.noisy_grid(w, h, seed=w) for w, h in sizes]
    nv, nf = [p[0].shape[0] for p in parts], [p[1].shape[0] for p in parts]
    base = np.concatenate([[0], np.cumsum(nv)])
    V, F = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] + np.int32(b) for p, b in zip(parts, base)])
    print(f"counts for itself {sum(nv)}", flush=True)
    for part in (0.55, 0.2):  # one round that its budget binds a little; several
        target = [max(int(n * part), 1) for n in nv]
        st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, target)
        ref = oracle.decimate_batch(V, F, nv, nf, target)
        assert list(nvo) == list(ref["nv"]) and list(nfo) == list(ref["nf"])
        assert_same_result(st, vo, fo, cid, ref)
    if len(parts) > 1:
        return
    ctx.set_placement(pk.PICASSO_PLACE_INVERSE, 1e-3)
    try:
        st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target[0])
        assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target[0], placement=1, rcond_min=1e-3))
    finally:
        ctx.set_placement(pk.PICASSO_PLACE_MEAN)


def test_statistics_and_timing_options_do_not_change_the_result(pk, ctx, oracle):
    """The per-round statistics agree with the oracle's bookkeeping; stage events and the kernel's
    launch events are measurement only."""
    V, F = meshgen.icosphere(5, seed=3)
    N, target = V.shape[0], V.shape[0] // 6
    ref = oracle.decimate(V, F, target)
    for stage, every in ((0, 0), (1, 0), (0, 1), (1, 2)):
        ctx.set_option(pk.PICASSO_OPT_STAGE_TIMING, stage)
        ctx.set_option(pk.PICASSO_OPT_KERNEL_TIMING, every)
        try:
            for k in range(pk.PICASSO_KERNEL_COUNT):
                ctx.picasso_kernel_timing(k, reset=True)
            st_ = pk.picasso_stats()
            for _ in range(3):
                st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target, stats=st_)
                assert_same_result(st, vo, fo, cid, ref)
            d = st_.as_dict()
            assert d["rounds"] == ref["rounds"] and d["nv_out"] == target and d["nf_out"] == ref["facets"].shape[0]
            assert d["nv"][0] == N and d["nf"][0] == F.shape[0] and d["ne"][0] == oracle.edges(F).shape[0]
            assert all(d["nv"][r + 1] == d["nv"][r] - d["nsel"][r] for r in range(d["rounds"] - 1))
            assert d["nv"][-1] - d["nsel"][-1] == target and d["ms_total"] > 0
            if stage:
                assert sum(sum(r.values()) for r in d["ms_stage"]) > 0
            timed_calls = {0: 0, 1: 3, 2: 2}[every]   # of the three calls above
            for k in range(pk.PICASSO_KERNEL_COUNT):
                kt = ctx.picasso_kernel_timing(k, reset=True)
                per_call = 1 if k in (pk.PICASSO_KERNEL_QUADRIC_ROWS, pk.PICASSO_KERNEL_SORT_INCIDENCE) else d["rounds"]
                assert kt["launches"] == timed_calls * per_call, (k, kt)
                if every:
                    assert kt["ms_total"] > 0 and kt["bytes_total"] > 0
                assert ctx.picasso_kernel_timing(k)["launches"] == 0           # the reset took
            with pytest.raises(pk.PicassoError):
                ctx.picasso_kernel_timing(pk.PICASSO_KERNEL_COUNT)
        finally:
            ctx.set_option(pk.PICASSO_OPT_STAGE_TIMING, 0)
            ctx.set_option(pk.PICASSO_OPT_KERNEL_TIMING, 0)


def test_vertices_of_medium_degree(ctx, oracle):
    """Cones whose apex has 17 to 130 facets: per-vertex groups of the sorts between the register
    network (up to 16 keys), the in-place insertion (up to 64) and the radix fallback beyond."""
    rng = np.random.default_rng(4)
    Vs, Fs = [], []
    base = 0
    for d in (3, 15, 16, 17, 31, 32, 33, 63, 64, 65, 96, 130) * 3:
        ang = np.linspace(0.0, 2.0 * np.pi, d, endpoint=False)
        ring = np.stack([np.cos(ang), np.sin(ang), np.zeros(d)], axis=1) * rng.uniform(0.5, 2.0)
        apex = np.array([[0.0, 0.0, rng.uniform(0.2, 1.5)]])
        P = np.concatenate([apex, ring]) + rng.normal(scale=0.01, size=(d + 1, 3)) + rng.uniform(-50, 50, size=(1, 3))
        tri = np.array([[0, 1 + i, 1 + (i + 1) % d] for i in range(d)])
        Vs.append(P.astype(np.float32))
        Fs.append(tri + base)
        base += d + 1
    # The cones come first (low indices) in a mesh of about 2^17 vertices: then the sorts' per-bucket
    # radix pass ends exactly at the lower vertex's bits, and an apex's edges (facets) form one group.
    room = meshgen.config("room115k")
    Vs.append(room["verts"])
    Fs.append(room["facets"] + base)
    V = np.concatenate(Vs)
    F = np.concatenate(Fs).astype(np.int32)
    assert 1 << 16 < V.shape[0] <= 1 << 17
    Q = ctx.picasso_vertex_quadrics(dev(V), dev(F)).cpu().numpy()
    assert np.array_equal(Q.view(np.uint32), oracle.vertex_quadrics(V, F).view(np.uint32))
    E, cost = ctx.picasso_edge_costs(dev(V), dev(F))
    assert np.array_equal(E.cpu().numpy(), oracle.edges(F))
    for frac in (0.7, 0.3):
        target = int(V.shape[0] * frac)
        st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
        assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))


def test_two_contexts_on_two_host_threads(pk, oracle):
    """Contexts share nothing: two host threads, each with a context, a stream and options of its
    own, decimate different meshes at the same time and each result matches the oracle's."""
    import threading
    room = meshgen.config("room115k")
    jobs = [
        dict(V=room["verts"], F=room["facets"], target=int(room["target"][0]), opts={}),
        dict(V=None, F=None, target=None, opts=dict(placement=1, rcond_min=1e-3, absorb=True, shuffle_seed=77)),
    ]
    jobs[1]["V"], jobs[1]["F"] = meshgen.icosphere(6, seed=2, jitter=0.05)
    jobs[1]["target"] = jobs[1]["V"].shape[0] // 5
    for j in jobs:
        j["ref"] = oracle.decimate(j["V"], j["F"], j["target"], **j["opts"])
        j["ctx"] = pk.Context(200_000, 400_000, 4, device=0)
        j["stream"] = torch.cuda.Stream()
        j["dV"], j["dF"] = dev(j["V"]), dev(j["F"])
        j["out"], j["err"] = [], None
    c1 = jobs[1]["ctx"]
    c1.set_placement(pk.PICASSO_PLACE_INVERSE, 1e-3)
    c1.set_option(pk.PICASSO_OPT_ABSORB, 1)
    c1.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, 77)
    torch.cuda.synchronize()
    start = threading.Barrier(2)

    def work(j):
        try:
            with torch.cuda.stream(j["stream"]):
                start.wait(timeout=30)
                for _ in range(20):
                    j["out"].append(j["ctx"].picasso_decimate(j["dV"], j["dF"], j["target"], stream=j["stream"]))
        except Exception as e:  # noqa: BLE001 -- reported by the main thread below
            j["err"] = e

    threads = [threading.Thread(target=work, args=(j,)) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
        assert not t.is_alive()
    torch.cuda.synchronize()
    try:
        for j in jobs:
            assert j["err"] is None, j["err"]
            assert len(j["out"]) == 20
            for st, vo, fo, cid in j["out"]:
                assert_same_result(st, vo, fo, cid, j["ref"])
    finally:
        for j in jobs:
            j["ctx"].close()


def test_ten_million_vertices(pk, oracle):
    """10.2 M vertices, 20.5 M facets, 61 M half-edges (a 6 GiB workspace): every index that is
    multiplied by a record size goes beyond 2^31 bytes, the sorts partition on 16 bits and more over
    tens of thousands of tiles.  About 15 s of oracle time."""
    V, F = meshgen.noisy_grid(3200, 3200, seed=5, noise=0.004)
    target = V.shape[0] // 4
    print(f"large mesh: N={V.shape[0]} F={F.shape[0]} -> {target}", flush=True)
    c = pk.Context(V.shape[0], F.shape[0], 1, device=0)
    try:
        st, vo, fo, cid = c.picasso_decimate(dev(V), dev(F), target)
        print("decimated; oracle running", flush=True)
        assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))
    finally:
        c.close()


def test_host_wait_by_stream_synchronisation_or_by_watching_pinned_memory(pk, ctx, oracle):
    """PICASSO_OPT_HOST_POLL only changes how the host learns that a round's selection is done."""
    V, F = meshgen.icosphere(5, seed=11, jitter=0.05)
    target = V.shape[0] // 7
    ref = oracle.decimate(V, F, target)
    b = meshgen.config("grid64")
    for poll in (0, 1, 2, 0, 50, 1):   # 2 and 50 us: the watch gives up and the stream is synchronised instead
        ctx.set_option(pk.PICASSO_OPT_HOST_POLL, poll)
        try:
            for _ in range(5):
                st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
                assert_same_result(st, vo, fo, cid, ref)
            st, vo, fo, cid = ctx.picasso_decimate(dev(b["verts"]), dev(b["facets"]), int(b["target"][0]))
            assert_same_result(st, vo, fo, cid, oracle.decimate(b["verts"], b["facets"], int(b["target"][0])))
        finally:
            ctx.set_option(pk.PICASSO_OPT_HOST_POLL, 1)
    with pytest.raises(pk.PicassoError):
        ctx.set_option(pk.PICASSO_OPT_HOST_POLL, -1)


@pytest.mark.parametrize("batch", [1, 16])
def test_kernels_queued_ahead_of_the_hosts_look(pk, ctx, oracle, batch):
    """PICASSO_OPT_LAUNCH_AHEAD: in rounds whose budget cannot bind, the contraction and facet kernels
    are queued behind the selection before the host knows its outcome.  With one sub-round per
    batch the selection is not finished at the first look, so the queued kernels must do nothing and
    be queued again; results equal the oracle's either way, on a single mesh and on a batch."""
    V, F = meshgen.icosphere(5, seed=13, jitter=0.05)
    target = V.shape[0] // 9                      # four rounds, the first three far from the budget
    ref = oracle.decimate(V, F, target)
    assert ref["rounds"] >= 3
    c5 = meshgen.config("batch16x60k")
    nv, nf, tg = c5["nv"][:3], c5["nf"][:3], c5["target"][:3]
    Vb, Fb = c5["verts"][: nv.sum()], c5["facets"][: nf.sum()]
    refb = oracle.decimate_batch(Vb, Fb, nv, nf, tg)
    ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, batch)
    try:
        for ahead in (1, 0, 1):
            ctx.set_option(pk.PICASSO_OPT_LAUNCH_AHEAD, ahead)
            st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
            assert_same_result(st, vo, fo, cid, ref)
            st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(Vb), dev(Fb), nv, nf, tg)
            assert st == refb["status"]
            assert np.array_equal(cid.cpu().numpy(), refb["cluster_id"])
            assert np.array_equal(fo.cpu().numpy(), refb["facets"])
            assert np.array_equal(vo.cpu().numpy().view(np.uint32), refb["verts"].view(np.uint32))
    finally:
        ctx.set_option(pk.PICASSO_OPT_LAUNCH_AHEAD, 1)
        ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, 16)


@pytest.mark.parametrize("fixture", ["two_quads_hand.json", "duplicate_facets_hand.json", "fan_two_runs_hand.json"])
def test_hand_worked_fixtures_on_the_gpu(pk, ctx, fixture):
    """The hand-worked examples under tests/golden (values written out by hand from Alg. 2 and the
    supplementary's placement and quadric equations) compared with the HIP path directly: output
    positions, the facet list in order and winding, and the cluster map."""
    import json
    import os
    fx = json.load(open(os.path.join(os.path.dirname(__file__), "golden", fixture)))
    V = np.asarray(fx["verts"], np.float32)
    F = np.asarray(fx["facets"], np.int32)
    for case in fx["cases"]:
        print(f"fixture {fixture} target={case['target']}", flush=True)
        ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, case.get("max_rounds", -1))
        try:
            st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), case["target"])
        finally:
            ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, -1)
        assert st in (0, 1)
        assert vo.cpu().numpy().tolist() == case["verts_out"]
        assert fo.cpu().numpy().reshape(-1, 3).tolist() == case["facets_out"]
        assert cid.cpu().numpy().tolist() == case["cluster_id"]


def test_budget_search_refuses_sizes_it_was_not_launched_for(pk, ctx, oracle):
    """The per-mesh budget step is launched for up to 4,096 or 32,768 pairs a mesh.  Forced (test hook) to 4 x 1,024 on a mesh that forms more than 4096 pairs, the kernel must make the call fail with
    PICASSO_ERR_INTERNAL rather than return with the budget not applied; the context stays usable."""
    V, F = meshgen.noisy_grid(130, 120, seed=17)          # 15,600 vertices: about 7,000 pairs per round
    target = int(V.shape[0] * 0.62)                       # the budget binds in the first round
    ctx.set_option(pk.PICASSO_OPT_TRUNC_WIDTH, 4)
    try:
        print("budget search, width forced to 4", flush=True)
        with pytest.raises(pk.PicassoError) as ei:
            ctx.picasso_decimate(dev(V), dev(F), target)
        assert ei.value.status == pk.PICASSO_ERR_INTERNAL
        # a mesh that fits the forced width is unaffected
        Vs, Fs = meshgen.noisy_grid(40, 40, seed=3)
        st, vo, fo, cid = ctx.picasso_decimate(dev(Vs), dev(Fs), 1000)
        assert_same_result(st, vo, fo, cid, oracle.decimate(Vs, Fs, 1000))
    finally:
        ctx.set_option(pk.PICASSO_OPT_TRUNC_WIDTH, 0)
    st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), target)
    assert_same_result(st, vo, fo, cid, oracle.decimate(V, F, target))
    with pytest.raises(pk.PicassoError):
        ctx.set_option(pk.PICASSO_OPT_TRUNC_WIDTH, 5)


def test_degenerated_vertices_dropped(pk, ctx, ctx16k, oracle):
    """PICASSO_OPT_DROP_DEGENERATED: output vertices that no output facet refers to are dropped; against the
    hand-worked fixture, and against the oracle's post-processing on soups, a room, a batch and a call
    that runs zero rounds; replace / mapping (both entry points) take the -1 cluster ids."""
    import json
    import os
    fx = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "drop_degenerated_hand.json")))

    def check(c, V, F, target, ref):
        st, vo, fo, cid = c.picasso_decimate(dev(V), dev(F), target)
        assert vo.shape[0] == ref["verts"].shape[0]
        assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))
        assert np.array_equal(fo.cpu().numpy(), ref["facets"]) and np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
        return cid, vo.shape[0]

    for c in (ctx, ctx16k):
        c.set_option(pk.PICASSO_OPT_DROP_DEGENERATED, 1)
    try:
        V = np.asarray(fx["verts"], np.float32)
        F = np.asarray(fx["facets"], np.int32)
        for case in fx["cases"]:
            print(f"drop degenerated: fixture target={case['target']}", flush=True)
            st, vo, fo, cid = ctx.picasso_decimate(dev(V), dev(F), case["target"])
            assert vo.cpu().numpy().tolist() == case["dropped"]["verts_out"]
            assert fo.cpu().numpy().reshape(-1, 3).tolist() == case["dropped"]["facets_out"]
            assert cid.cpu().numpy().tolist() == case["dropped"]["cluster_id"]
            rep, mp = ctx.picasso_replace_mapping(cid, vo.shape[0])
            assert rep.cpu().numpy().tolist() == case["dropped"]["replace"]
            assert mp.cpu().numpy().tolist() == case["dropped"]["mapping"]
            rep2, mp2 = torch.zeros_like(rep), torch.zeros_like(mp)
            status = torch.zeros(1, dtype=torch.int32, device="cuda:0")
            assert pk.picasso_replace_mapping_static(cid, vo.shape[0], rep2, mp2, status) == pk.PICASSO_OK
            torch.cuda.synchronize()
            assert int(status.item()) == 0 and torch.equal(rep, rep2) and torch.equal(mp, mp2)
        rng = np.random.default_rng(8)
        for k in range(6):
            nv = int(rng.integers(10, 400))
            V = rng.normal(size=(nv, 3)).astype(np.float32)
            F = rng.integers(0, max(3, nv * 2 // 3), size=(int(rng.integers(4, 600)), 3)).astype(np.int32)
            target = max(2, nv // int(rng.integers(2, 6)))
            print(f"drop degenerated: soup {k} nv={nv} target={target}", flush=True)
            check(ctx, V, F, target, oracle.drop_unreferenced(oracle.decimate(V, F, target)))
        V, F = meshgen.room_scene(5, room=(3.0, 2.0, 1.5), n_boxes=6, spacing=0.04)
        V = np.concatenate([V, rng.normal(size=(100, 3)).astype(np.float32)])          # 100 vertices in no facet
        for target in (V.shape[0] + 5, V.shape[0] // 3, 50):                            # zero rounds, a few, many
            print(f"drop degenerated: room N={V.shape[0]} target={target}", flush=True)
            cid, n_out = check(ctx, V, F, target, oracle.drop_unreferenced(oracle.decimate(V, F, target)))
            assert int((cid[-100:] == -1).sum()) == 100
        parts = [meshgen.noisy_grid(30, 22, seed=1), meshgen.icosphere(3, seed=2), meshgen.noisy_grid(12, 12, seed=3)]
        parts[0] = (np.concatenate([parts[0][0], rng.normal(size=(7, 3)).astype(np.float32)]), parts[0][1])
        nv = [p[0].shape[0] for p in parts]
        nf = [p[1].shape[0] for p in parts]
        off = np.cumsum([0] + nv)
        V = np.concatenate([p[0] for p in parts])
        F = np.concatenate([p[1] + off[i] for i, p in enumerate(parts)]).astype(np.int32)
        tg = [200, 700, 4]
        print("drop degenerated: batch", flush=True)
        st, vo, fo, cid, nvo, nfo = ctx16k.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
        rb = oracle.decimate_batch(V, F, nv, nf, tg)
        ref = oracle.drop_unreferenced(rb, nv=rb["nv"])
        assert nvo.tolist() == ref["nv"].tolist() and nfo.tolist() == rb["nf"].tolist()
        assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))
        assert np.array_equal(fo.cpu().numpy(), ref["facets"]) and np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
    finally:
        for c in (ctx, ctx16k):
            c.set_option(pk.PICASSO_OPT_DROP_DEGENERATED, 0)


@pytest.mark.parametrize("flat", [False, True])
def test_budget_of_long_runs_in_a_batch(pk, oracle, flat):
    """Two meshes of a batch form more pairs than one workgroup selects from (one keeps a single pair, one most of
    them), next to meshes that form few; with distinct costs, and with nothing but ties."""
    make = (lambda w, h, seed: meshgen.flat_grid(w, h, spacing=0.25)) if flat else (lambda w, h, seed: meshgen.noisy_grid(w, h, seed=seed))
    parts = [make(30, 22, 1), make(330, 270, 2), make(12, 9, 3), make(300, 301, 4)]
    nv, nf = [p[0].shape[0] for p in parts], [p[1].shape[0] for p in parts]
    off = np.cumsum([0] + nv)
    V = np.concatenate([p[0] for p in parts])
    F = np.concatenate([p[1] + off[i] for i, p in enumerate(parts)]).astype(np.int32)
    tg = [nv[0] - 40, nv[1] - 1, nv[2], nv[3] - 30000]
    c = pk.Context(V.shape[0], F.shape[0], len(parts), device=0)
    try:
        st, vo, fo, cid, nvo, nfo = c.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
        ref = oracle.decimate_batch(V, F, nv, nf, tg)
        assert st == ref["status"] and nvo.tolist() == ref["nv"].tolist() and nfo.tolist() == ref["nf"].tolist()
        assert np.array_equal(cid.cpu().numpy(), ref["cluster_id"])
        assert np.array_equal(fo.cpu().numpy(), ref["facets"])
        assert np.array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))
    finally:
        c.close()


def test_budget_of_a_long_run_behind_more_meshes_than_a_grid_has_rows(pk, oracle):
    """66,000 two-facet meshes and, behind them, one of 38,000 pairs whose budget binds."""
    small, big = meshgen.noisy_grid(2, 2, seed=1), meshgen.noisy_grid(290, 285, seed=2)
    k, (v, f) = 66000, small
    nv, nf = [v.shape[0]] * k + [big[0].shape[0]], [f.shape[0]] * k + [big[1].shape[0]]
    V = np.concatenate([np.tile(v, (k, 1)), big[0]])
    F = np.concatenate([(f[None] + (4 * np.arange(k))[:, None, None]).reshape(-1, 3), big[1] + 4 * k]).astype(np.int32)
    tg = [4] * k + [big[0].shape[0] - 36000]
    ctx = pk.Context(V.shape[0], F.shape[0], len(nv), device=0)
    try:
        print(f"{len(nv)} meshes, {V.shape[0]} vertices", flush=True)
        st, vo, fo, cid, nvo, nfo = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, tg)
    finally:
        ctx.close()
    ref = oracle.decimate(*big, tg[-1])
    assert st == ref["status"] == 0 and nvo.tolist() == tg and int(nfo[-1]) == ref["facets"].shape[0]
    assert np.array_equal(vo.cpu().numpy()[4 * k:].view(np.uint32), ref["verts"].view(np.uint32))
    assert np.array_equal(fo.cpu().numpy()[2 * k:], ref["facets"] + 4 * k)
    assert np.array_equal(cid.cpu().numpy()[4 * k:], ref["cluster_id"] + 4 * k)
    assert np.array_equal(vo.cpu().numpy()[: 4 * k], V[: 4 * k]) and np.array_equal(fo.cpu().numpy()[: 2 * k], F[: 2 * k])
