"""The gradient of the fuzzy coefficients where a row's lanes lie in one wave: rows of 4 to 64 lanes, powers of two (whose lanes sum several
components together) and not, whole and ragged last packs, component counts at the edges of the groups of four, eight, twelve and sixteen and
over several passes; facets that leave waves incomplete.  Against the fp64 oracle with the bounds of test_gpu_conv."""
import numpy as np
import pytest
from scipy.special import softmax

from test_gpu_conv import _close, _gw_terms, ctx, dev, pk  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C", [9, 16, 31, 32, 36, 64, 125, 128, 253, 256])
@pytest.mark.parametrize("T", [1, 3, 4, 5, 8, 9, 11, 12, 13, 16, 17, 27])
def test_gradient_of_the_coefficients(pk, ctx, oracle, C, T):  # noqa: F811
    n, nF = 301, 517
    print(f"coefficients' gradient C={C} T={T}", flush=True)
    rng = np.random.default_rng(C * 100 + T)
    F = rng.integers(0, n, (nF, 3)).astype(np.int32)
    gx = rng.normal(size=(n, C)).astype(np.float32)
    y = rng.normal(size=(nF, C)).astype(np.float32)
    w = rng.normal(size=(T, C)).astype(np.float32)
    pi = softmax(rng.normal(size=(nF, T)), axis=1).astype(np.float32)
    off, _ = ctx.picasso_vertex_corner_csr(dev(F), n)
    want, bound = oracle.f2v_backward(gx, y, pi, w, F), oracle.f2v_backward(np.abs(gx), np.abs(y), pi, np.abs(w), F)
    got = ctx.picasso_f2v_backward(dev(gx), dev(y), dev(pi), dev(w), dev(F), off)
    for g, r, s, k, what in zip(got, want, bound, (T + 8, _gw_terms(nF, 6), 6 * C), ("gy", "gw", "gpi")):
        _close(g, r, k, s, what)
