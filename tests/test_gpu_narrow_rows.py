"""Convolutions of up to 8 channels, whose rows have a lane each: every channel count, component counts at the edges of their groups of
four, rows with as many items as one lane walks, one more (the whole wave's) and several such rows in a wave, counts of rows that leave
waves and workgroups incomplete; against the fp64 oracle with the bounds of test_gpu_conv."""
import numpy as np
import pytest
import torch
from scipy.special import softmax

from test_gpu_conv import _close, _gw_terms, ctx, dev, pk  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def _fans(sizes, n):
    """A fan of so many facets at each of the first vertices, over n vertices; the last few are unused."""
    rim = n - 7 - len(sizes)
    F = []
    for hub, m in enumerate(sizes):
        k = np.arange(m) * (2 * hub + 1)
        F.append(np.stack([np.full(m, hub), len(sizes) + k % rim, len(sizes) + (k + 1) % rim], 1))
    F = np.concatenate(F).astype(np.int32)
    return F[np.random.default_rng(n).permutation(len(F))]


@pytest.mark.parametrize("C,T", [(1, 1), (2, 4), (3, 5), (4, 8), (5, 9), (6, 6), (7, 12), (8, 13), (8, 16), (4, 16), (6, 3)])
@pytest.mark.parametrize("sizes,n", [([64, 65, 3, 700, 66, 1, 63], 300), ([257], 1025), ([1] * 60, 129)])
def test_narrow_rows(pk, ctx, oracle, C, T, sizes, n):  # noqa: F811
    F = _fans(sizes, n)
    nF = F.shape[0]
    print(f"narrow rows C={C} T={T} N={n} F={nF}", flush=True)
    rng = np.random.default_rng(C * 100 + T)
    x, gx = rng.normal(size=(2, n, C)).astype(np.float32)
    y, gy = rng.normal(size=(2, nF, C)).astype(np.float32)
    w3, w = rng.normal(size=(3, C)).astype(np.float32), rng.normal(size=(T, C)).astype(np.float32)
    pi = softmax(rng.normal(size=(nF, T)), axis=1).astype(np.float32)
    lv = rng.integers(1, 4, nF).astype(np.int32)
    off, cor = ctx.picasso_vertex_corner_csr(dev(F), n)
    deg = int(np.bincount(F.reshape(-1), minlength=n).max())
    for level in (lv, None):
        lr = lv if level is not None else np.ones(nF, np.int32)
        got = ctx.picasso_v2f_backward(dev(gy), dev(x), dev(F), None if level is None else dev(level), dev(w3), off, cor)
        ref, bar = oracle.v2f_backward(gy, x, F, lr, w3), oracle.v2f_backward(np.abs(gy), np.abs(x), F, lr, np.abs(w3))
        _close(got[0], ref[0], 4 * deg, bar[0], "v2f gx")
        _close(got[1], ref[1], _gw_terms(nF, 4), bar[1], "v2f gw")
    got = ctx.picasso_f2v_forward(dev(y), dev(pi), dev(w), off, cor, n)
    _close(got, oracle.f2v_forward(y, pi, w, F, n), (T + 2) * deg, oracle.f2v_forward(np.abs(y), pi, np.abs(w), F, n), "f2v")
    ref, bar = oracle.f2v_backward(gx, y, pi, w, F), oracle.f2v_backward(np.abs(gx), np.abs(y), pi, np.abs(w), F)
    for want in (True, False):
        got = ctx.picasso_f2v_backward(dev(gx), dev(y), dev(pi), dev(w), dev(F), off, want_gpi=want)
        _close(got[0], ref[0], T + 8, bar[0], "f2v gy")
        _close(got[1], ref[1], _gw_terms(nF, 6), bar[1], "f2v gw")
        if want:
            _close(got[2], ref[2], 6 * C, bar[2], "f2v gpi")


@pytest.mark.parametrize("C,T", [(3, 6), (6, 6), (8, 5)])
def test_narrow_rows_at_any_4_byte_address(pk, ctx, oracle, C, T):  # noqa: F811
    """Arrays that begin 4, 8 and 12 bytes behind a 16-byte line give what aligned ones give, bit for bit."""
    F = _fans([64, 65, 3, 200], 500)
    n, nF = 500, F.shape[0]
    rng = np.random.default_rng(C)
    host = [rng.normal(size=s).astype(np.float32) for s in ((n, C), (n, C), (nF, C), (nF, C), (3, C), (T, C))]
    pi = softmax(rng.normal(size=(nF, T)), axis=1).astype(np.float32)
    off, cor = ctx.picasso_vertex_corner_csr(dev(F), n)

    def calls(shift):
        def put(a):
            b = torch.zeros(a.size + 4, device="cuda:0")
            b[shift:shift + a.size] = torch.from_numpy(a.reshape(-1)).to("cuda:0")
            return b[shift:shift + a.size].reshape(a.shape)
        x, gx, y, gy, w3, w = map(put, host)
        p = put(pi)
        out = [*ctx.picasso_v2f_backward(gy, x, dev(F), None, w3, off, cor), ctx.picasso_f2v_forward(y, p, w, off, cor, n),
               *ctx.picasso_f2v_backward(gx, y, p, w, dev(F), off)]
        return [t.cpu().numpy().view(np.uint32) for t in out]

    want = calls(0)
    for shift in (1, 2, 3):
        for a, b in zip(calls(shift), want):
            np.testing.assert_array_equal(a, b)
