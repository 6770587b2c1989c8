"""The list of the budget step by the whole chip (budget_range_kernel) holds the pairs that its sample points at, up to the most pairs with which a call takes this way: the
same sample, range and list in numpy, on the pairs that the oracle forms.  (The kernels' results are the same where the list overflows, by another way.)"""
import os
import re

import numpy as np
import pytest

from paper_2103_15076_amd import meshgen

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2103_15076_amd", "csrc")
NONE = np.uint32(0xFFFFFFFF)


def constant(name, file="picasso.hip"):
    with open(os.path.join(CSRC, file)) as f:
        return eval(re.search(r"\b%s = ([^,;]+)[,;]" % name, f.read()).group(1).replace("BUDGET_THREADS", "1024"))


def formed_pairs(oracle, V, F):
    """Cost key of every pair that the matching forms, at its lower vertex."""
    E = oracle.edges(F)
    _, key = oracle.edge_costs(V, oracle.vertex_quadrics(V, F), E)
    sel, _ = oracle.select(E, key, len(V), len(V))
    pcost = np.full(len(V), NONE, np.uint32)
    pcost[E[sel].min(1)] = key[sel]
    return pcost


def listed(pcost, keep):
    nv, few = len(pcost), 1 << 16
    lanes = np.arange(4 * 1024 if nv > few else 1024, dtype=np.int64)
    place = (nv * lanes >> (12 if nv > few else 10)) & ~3
    at = (place[:, None] + np.arange(4)).reshape(-1)
    sample = pcost[at[at < nv]]
    drop = np.uint32(18)  # bits that the range's ends leave open
    sample = np.sort(sample[sample != NONE] >> drop).astype(np.int64)
    n, total = int((pcost != NONE).sum()), len(sample)
    rank, margin = np.float32(total) * np.float32(keep) / np.float32(n), np.float32(3) * np.sqrt(np.float32(total)) + np.float32(4)
    first, last = int(rank - margin) if rank > margin else 0, min(int(rank + margin), total + 1)
    lo = int(sample[first - 1]) << int(drop) if first > 0 else 0
    hi = (int(sample[last - 1]) << int(drop) | (1 << int(drop)) - 1) if 0 < last <= total else 0xFFFFFFFE
    key = pcost[pcost != NONE].astype(np.int64)
    below, count = int((key < lo).sum()), int(((key >= lo) & (key <= hi)).sum())
    assert below < keep <= below + count, "the sample has missed the pair"
    return count


@pytest.mark.parametrize("mesh", ["lattice", "room"])
def test_the_list_holds_the_most_pairs(oracle, mesh):
    most = 2 * constant("BUDGET_CHIP_MAX")  # vertices
    if mesh == "lattice":
        side = int(most ** 0.5)
        V, F = meshgen.noisy_grid(side, most // side, seed=3)
    else:
        V, F = meshgen.room_scene_sized(5, int(0.99 * most))[:2]
    assert 0.95 * most < len(V) <= most + 1
    pcost = formed_pairs(oracle, V, F)
    n, cap = int((pcost != NONE).sum()), constant("BUDGET_LIST", "decimate_kernels.h")
    assert cap == 32 * 1024
    for share in np.arange(0.025, 1, 0.025):
        assert listed(pcost, int(share * n)) <= cap, share
