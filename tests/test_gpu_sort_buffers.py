"""What else the sorts' buffers are lent to: a filter gradient whose partial sums fill them leaves nothing behind that a decimation, or the
same gradient again, on that context would notice."""
import numpy as np
import pytest
from scipy.special import softmax

from paper_2103_15076_amd import meshgen
from test_gpu_facet_rounds import dev, pk, same  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,T", [(64, 16), (257, 6), (300, 16)])
def test_partial_sums_fill_the_sort_buffers(pk, oracle, C, T):  # noqa: F811
    V, F = meshgen.noisy_grid(61, 47, seed=C)
    N, nF = len(V), len(F)
    rng = np.random.default_rng(C)
    gx, y = rng.normal(size=(N, C)).astype(np.float32), rng.normal(size=(nF, C)).astype(np.float32)
    pi, w = softmax(rng.normal(size=(nF, T)), axis=1).astype(np.float32), rng.normal(size=(T, C)).astype(np.float32)
    ctx = pk.Context(N, nF, 1, device=0)
    off, _ = ctx.picasso_vertex_corner_csr(dev(F), N)
    ref = oracle.decimate(V, F, N // 3)
    grads = []
    for _ in range(2):
        same(ctx.picasso_decimate(dev(V), dev(F), N // 3), ref)
        grads.append([g.cpu().numpy() for g in ctx.picasso_f2v_backward(dev(gx), dev(y), dev(pi), dev(w), dev(F), off)])
    for a, b in zip(*grads):
        np.testing.assert_array_equal(a, b)
    want, size = oracle.f2v_backward(gx, y, pi, w, F)[1], oracle.f2v_backward(np.abs(gx), np.abs(y), pi, np.abs(w), F)[1]
    assert np.all(np.abs(grads[0][1] - want) <= (nF + 16) * 2.0 ** -24 * size)  # (nF + 16 roundings at the most, however the sum is split)
