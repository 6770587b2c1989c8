"""Statistics are those of the rounds that the same call runs without them: by facets, where a selection hands back to the host by the number of
live copies of its edges, while the distinct edges, which such a round does not list, are counted for the statistics."""
import numpy as np
import pytest

from test_gpu_facet_rounds import dev, lattice, pk, same  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_facets", [1, 257, 6000, (1 << 20) + 3])
@pytest.mark.parametrize("stages", [0, 1])
def test_distinct_edges_of_every_round(pk, oracle, n_facets, stages):  # noqa: F811
    V, F = lattice(n_facets, 5, 0.3, 0.1)
    target = max(1, len(V) // 4)
    ctx = pk.Context(len(V), len(F), 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_STAGE_TIMING, stages)
    st = pk.picasso_stats()
    same(ctx.picasso_decimate(dev(V), dev(F), target, stats=st), oracle.decimate(V, F, target))
    d = st.as_dict()
    for r in range(d["rounds"]):
        before = oracle.decimate(V, F, target, max_rounds=r)["facets"] if r else F
        assert d["ne"][r] == len(oracle.edges(before)) and d["nsel"][r] > 0
    assert d["ms_total"] > 0


def test_sub_rounds_are_those_by_facets(pk, oracle):  # noqa: F811
    """About 3,000 distinct edges are live behind the first sub-round, which the tail takes, and in facets without order twice as many copies,
    which it hands back once."""
    V, F = lattice(6000, 5)
    F = F[np.random.default_rng(0).permutation(len(F))]
    ctx = pk.Context(len(V), len(F), 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_SUBROUND_BATCH, 1)
    ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, 1)
    launched = []
    for absorb in (0, 1):  # (line 11 needs the edges sorted)
        ctx.set_option(pk.PICASSO_OPT_ABSORB, absorb)
        st = pk.picasso_stats()
        ctx.picasso_decimate(dev(V), dev(F), 1, stats=st)
        assert st.ne[0] == len(oracle.edges(F))
        launched.append(st.subrounds[0])
    assert launched == [4, 2]


def test_a_batch_of_sub_rounds_does_for_two_sided_surfaces(pk):  # noqa: F811
    """Every edge of which has four facets: five sub-rounds and the tail, which need not hand back."""
    V, F = lattice(79000, 9)
    F = np.concatenate([F, F[:, ::-1]])
    ctx = pk.Context(len(V), len(F), 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_MAX_ROUNDS, 1)
    st = pk.picasso_stats()
    ctx.picasso_decimate(dev(V), dev(F), 1, stats=st)
    assert st.subrounds[0] == 6
