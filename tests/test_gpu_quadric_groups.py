"""Vertex quadrics from the groups of the incidence sort, a lane per vertex: vertices of 0 to 16 facets (one lane sorts them), 17 to 64 (a
wave), one more (the whole bucket is sorted the other way) and more than a workgroup of 128 lanes keeps in LDS, buckets that end behind the last vertex, few and many keys to a bucket;
bit for bit against the oracle."""
import numpy as np
import pytest

from paper_2103_15076_amd import meshgen
from test_gpu_facet_rounds import dev, pk  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[], [1, 4, 7, 8, 9, 12, 15, 16], [16, 17, 18, 40, 63, 64], [17, 64, 65, 300], [3000]],
                         ids=["surface", "lane", "wave", "long", "beyond-lds"])
@pytest.mark.parametrize("w,h", [(53, 57), (300, 241), (700, 501)])
def test_vertices_of_any_number_of_facets(pk, oracle, sizes, w, h):  # noqa: F811
    V, F = meshgen.noisy_grid(w, h, seed=w)
    N = len(V)
    rng = np.random.default_rng(w + len(sizes))
    extra = []
    for k, m in enumerate(sizes):  # fans around vertices that had no facet, a few apart, in any order among the facets
        hubs = N + 5 * k + 40 * np.arange(20)
        rim = rng.integers(0, N, (20, m, 2))
        extra.append(np.concatenate([np.concatenate([np.full((m, 1), v), r], 1) for v, r in zip(hubs, rim)]))
    V = np.concatenate([V, rng.normal(size=(900, 3)).astype(np.float32)])  # (most of them without facets)
    F = np.concatenate([F] + extra).astype(np.int32)
    F = np.ascontiguousarray(F[rng.permutation(len(F))])
    print(f"quadrics N={len(V)} F={len(F)} {sizes}", flush=True)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    got = ctx.picasso_vertex_quadrics(dev(V), dev(F)).cpu().numpy()
    want = oracle.vertex_quadrics(V, F).astype(np.float32)
    np.testing.assert_array_equal(got.view(np.uint32), want.view(np.uint32))


def test_vertices_most_of_which_have_no_facet(pk, oracle):  # noqa: F811
    """Two buckets hold all keys, five times what fits LDS: 256 lanes sort them, not the 128 of buckets that hold as few as these do on average (549 us)."""
    V, F = meshgen.noisy_grid(60, 60, seed=60)
    V = np.concatenate([V, np.random.default_rng(1).normal(size=(300000, 3)).astype(np.float32)])
    v, f = dev(V), dev(F)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    got = ctx.picasso_vertex_quadrics(v, f).cpu().numpy()
    np.testing.assert_array_equal(got.view(np.uint32), oracle.vertex_quadrics(V, F).astype(np.float32).view(np.uint32))
    ctx.set_option(pk.PICASSO_OPT_KERNEL_TIMING, 1)
    ctx.picasso_kernel_timing(pk.PICASSO_KERNEL_QUADRIC_ROWS, reset=True)
    for _ in range(10):
        ctx.picasso_decimate(v, f, len(V) - 500)
    took = ctx.picasso_kernel_timing(pk.PICASSO_KERNEL_QUADRIC_ROWS, reset=True)
    assert took["launches"] == 10 and took["ms_total"] / 10 < 0.4, took
