"""Alg. 2 line 11's candidates queued behind the selection before the host has looked: budgets of which a round can take all, some and
too many, selections that hand back to the host (the candidates are then made again), several meshes; against the oracle, and with
nothing queued ahead."""
import numpy as np
import pytest

from test_gpu_facet_rounds import dev, lattice, pk, same  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [16, 1])
@pytest.mark.parametrize("seed", [0, 7])
@pytest.mark.parametrize("n_facets,keep", [(60, 0.3), (3000, 0.2), (3000, 0.45), (3000, 0.5), (3000, 0.7), (40000, 0.3)])
def test_candidates_of_one_mesh(pk, oracle, n_facets, keep, seed, batch):  # noqa: F811
    V, F = lattice(n_facets, 11 + seed)
    target = max(1, int(len(V) * keep))
    ctx = pk.Context(len(V), len(F), 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_ABSORB, 1)
    ctx.set_option(pk.PICASSO_OPT_SHUFFLE_SEED, seed)
    ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, batch)
    ref = oracle.decimate(V, F, target, absorb=True, shuffle_seed=seed)
    for ahead in (1, 0, 1):
        ctx.set_option(pk.PICASSO_OPT_LAUNCH_AHEAD, ahead)
        same(ctx.picasso_decimate(dev(V), dev(F), target), ref)


@pytest.mark.parametrize("keeps", [(0.3, 0.4, 0.5), (0.2, 0.9, 0.4), (0.1, 1.0, 0.6)])
def test_candidates_of_several_meshes(pk, oracle, keeps):  # noqa: F811
    parts = [lattice(n, k) for k, n in enumerate((5000, 900, 20000))]
    nv, nf = [len(v) for v, _ in parts], [len(f) for _, f in parts]
    base = np.concatenate([[0], np.cumsum(nv)])
    V = np.concatenate([v for v, _ in parts])
    F = np.concatenate([f + np.int32(base[k]) for k, (_, f) in enumerate(parts)])
    target = [max(1, int(n * k)) for n, k in zip(nv, keeps)]
    refs = [oracle.decimate(v, f, t, absorb=True) for (v, f), t in zip(parts, target)]
    nv_ref, nf_ref = [len(r["verts"]) for r in refs], [len(r["facets"]) for r in refs]
    first = np.concatenate([[0], np.cumsum(nv_ref)])  # (of a mesh's output vertices)
    ref = dict(status=max(r["status"] for r in refs), verts=np.concatenate([r["verts"] for r in refs]),
               facets=np.concatenate([r["facets"] + np.int32(first[k]) for k, r in enumerate(refs)]),
               cluster_id=np.concatenate([r["cluster_id"] + np.int32(first[k]) for k, r in enumerate(refs)]))
    ctx = pk.Context(len(V), len(F), 3, device=0)
    ctx.set_option(pk.PICASSO_OPT_ABSORB, 1)
    for ahead, batch in ((0, 16), (1, 16), (1, 1)):
        ctx.set_option(pk.PICASSO_OPT_LAUNCH_AHEAD, ahead)
        ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, batch)
        got = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, target)
        same(got, ref)
        assert list(got[4]) == nv_ref and list(got[5]) == nf_ref
