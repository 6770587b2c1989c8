"""Flat lattices, all of whose costs are equal: pairs form in a front that takes hundreds of sub-rounds to cross the mesh, with the edges in front of it
live all the while.  Against the oracle; the host looks seldom then, and no sub-round is left to a few workgroups."""
import time

import numpy as np
import pytest

from paper_2103_15076_amd import meshgen
from test_gpu_facet_rounds import dev, pk, same  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,keep", [(40, 30, 0.4), (150, 110, 0.3), (150, 110, 0.7), (900, 600, 0.6)])
@pytest.mark.parametrize("absorb", [0, 1])
def test_flat_lattice(pk, oracle, w, h, keep, absorb):  # noqa: F811
    V, F = meshgen.flat_grid(w, h)
    target = int(len(V) * keep)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_ABSORB, absorb)
    same(ctx.picasso_decimate(dev(V), dev(F), target), oracle.decimate(V, F, target, absorb=bool(absorb)))


def test_the_host_looks_seldom(pk):  # noqa: F811
    """Of 299 sub-rounds (as many as pairs need that each wait for the one in front of them) with up to 16 in a batch, the tails of the batches are few."""
    V, F = meshgen.flat_grid(200, 200)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, 1)
    for absorb in (0, 1):
        ctx.set_option(pk.PICASSO_OPT_ABSORB, absorb)
        st = pk.picasso_stats()
        ctx.picasso_decimate(dev(V), dev(F), len(V) // 4, stats=st)
        assert 250 < st.subrounds[0] < 299 + 30  # (the last 30 or so within the tail)


def test_rounds_by_facets_take_about_as_long_as_sorted_ones(pk):  # noqa: F811
    """(20 times as long while a few workgroups had all live edges; now no longer.)"""
    V, F = meshgen.flat_grid(200, 200)
    v, f = dev(V), dev(F)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, 1)
    took = []
    for absorb in (0, 1):  # (line 11 needs the edges sorted)
        ctx.set_option(pk.PICASSO_OPT_ABSORB, absorb)
        times = []
        for _ in range(5):
            t0 = time.perf_counter()
            ctx.picasso_decimate(v, f, len(V) // 4)
            times.append(time.perf_counter() - t0)
        took.append(min(times))
    assert took[0] < 4.0 * took[1], took
