"""The set in which a call finds repeated facets, at its fullest (just under a facet for every two slots) and with vertices numbered in no order, whose
facets crowd its low end: against the oracle, and in a time that says that no search walks through what is full, or comes back to it."""
import time

import numpy as np
import pytest

from test_gpu_facet_rounds import dev, lattice, pk, same  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _random_numbering(n_facets, seed, repeated):
    V, F = lattice(n_facets, seed, 0.3, repeated)
    rng = np.random.default_rng(seed)
    p = rng.permutation(len(V))
    inv = np.empty_like(p)
    inv[p] = np.arange(len(V))
    return V[p], inv[F[rng.permutation(len(F))]].astype(np.int32)


@pytest.mark.parametrize("n_facets", [8192, 1 << 18])
@pytest.mark.parametrize("repeated", [0.0, 0.1])
def test_crowded_low_end(pk, oracle, n_facets, repeated):  # noqa: F811
    V, F = _random_numbering(n_facets, 3, repeated)
    v, f = dev(V), dev(F)
    target = len(V) * 99 // 100
    ctx = pk.Context(len(V), len(F), 1, device=0)
    same(ctx.picasso_decimate(v, f, target), oracle.decimate(V, F, target))
    times = []
    for _ in range(5):
        t0 = time.perf_counter()
        ctx.picasso_decimate(v, f, target)
        times.append(time.perf_counter() - t0)
    assert min(times) < 4e-3, times  # (2^18 facets: 45 ms with one jump and steps along the line from there on, 0.4 now)


def test_crowded_vertices(pk, oracle):  # noqa: F811
    """20 k random facets on 1 k vertices, more to a vertex than there are places around it: keeping nearly all of them takes hardly longer than
    keeping 60 % (1.5 times as long when searches went on by equal strides)."""
    rng = np.random.default_rng(2)
    V, F = rng.standard_normal((1000, 3)).astype(np.float32), rng.integers(0, 1000, (20000, 3)).astype(np.int32)
    v, f = dev(V), dev(F)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    took = []
    for target in (950, 600):
        same(ctx.picasso_decimate(v, f, target), oracle.decimate(V, F, target))
        times = []
        for _ in range(30):
            t0 = time.perf_counter()
            ctx.picasso_decimate(v, f, target)
            times.append(time.perf_counter() - t0)
        took.append(sorted(times)[len(times) // 2])
    assert took[0] < 1.25 * took[1], took
