"""Meshes that want to lose vertices and have no edge to lose one by (every facet names one vertex three times, or there are none), in batches
whose other meshes contract: they are passed through with their facets as they came, as alone."""
import numpy as np
import pytest

from test_gpu_facet_rounds import dev, lattice, pk, same  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("absorb", [0, 1])  # (rounds by facets and of sorted edges)
@pytest.mark.parametrize("batch", [16, 1])
@pytest.mark.parametrize("keep", [0.7, 0.2])
def test_facets_of_a_mesh_without_edges_stay(pk, oracle, keep, batch, absorb):  # noqa: F811
    points = np.arange(9, dtype=np.float32).reshape(3, 3)
    parts = [lattice(700, 1), (points, np.array([[1, 1, 1], [1, 1, 1], [0, 0, 0]], np.int32)), lattice(3000, 2, 0.2, 0.1),
             (points[:2], np.zeros((0, 3), np.int32)), (points[:1], np.array([[0, 0, 0]], np.int32))]
    nv, nf = [len(v) for v, _ in parts], [len(f) for _, f in parts]
    base = np.concatenate([[0], np.cumsum(nv)])
    V = np.concatenate([v for v, _ in parts])
    F = np.concatenate([f + np.int32(base[k]) for k, (_, f) in enumerate(parts)])
    target = [max(1, int(n * keep)) for n in nv]
    refs = [oracle.decimate(v, f, t, absorb=bool(absorb)) for (v, f), t in zip(parts, target)]
    nv_ref, nf_ref = [len(r["verts"]) for r in refs], [len(r["facets"]) for r in refs]
    assert nf_ref[1] == 3 and nf_ref[4] == 1
    first = np.concatenate([[0], np.cumsum(nv_ref)])
    ctx = pk.Context(len(V), len(F), len(parts), device=0)
    ctx.set_option(pk.PICASSO_OPT_ABSORB, absorb)
    ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, batch)
    got = ctx.picasso_decimate_batch(dev(V), dev(F), nv, nf, target)
    assert list(got[4]) == nv_ref and list(got[5]) == nf_ref
    same(got, dict(status=max(r["status"] for r in refs), verts=np.concatenate([r["verts"] for r in refs]),
                   facets=np.concatenate([r["facets"].reshape(-1, 3) + np.int32(first[k]) for k, r in enumerate(refs)]),
                   cluster_id=np.concatenate([r["cluster_id"] + np.int32(first[k]) for k, r in enumerate(refs)])))
