"""Decimations whose outputs lie over their own inputs, against the oracle: rounds by rings read the facets where the caller has them until the call's last kernels."""
import numpy as np
import pytest

from paper_2103_15076_amd import meshgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_15076_amd
    return paper_2103_15076_amd


@pytest.mark.parametrize("which", ["facets_out", "cluster_id", "verts_out", "verts_out over verts", "cluster_id at the end"])
@pytest.mark.parametrize("side", [12, 150])
@pytest.mark.parametrize("drop", [0, 1])
def test_outputs_over_inputs(pk, oracle, which, side, drop):
    V, F = meshgen.noisy_grid(side, side, seed=side)
    n, m = len(V), len(F)
    ctx = pk.Context(n, m, 1, device=0)
    ctx.set_option(pk.PICASSO_OPT_DROP_DEGENERATED, drop)
    for keep in (0.7, 0.2):  # one round and several
        v, f = torch.from_numpy(V).cuda(), torch.from_numpy(F).cuda()
        room = torch.empty(3 * m + n, dtype=torch.int32, device="cuda:0")
        room[:3 * m] = f.reshape(-1)
        f = room[:3 * m].view(m, 3)
        over = {"facets_out": lambda: dict(facets_out=f), "cluster_id": lambda: dict(cluster_id=room[:n]),
                "verts_out": lambda: dict(verts_out=room[:3 * n].view(torch.float32).view(n, 3)), "verts_out over verts": lambda: dict(verts_out=v),
                "cluster_id at the end": lambda: dict(cluster_id=room[3 * m - 1:3 * m - 1 + n])}[which]()
        if 3 * n > 3 * m and which == "verts_out":
            pytest.skip("fewer facets than vertices")
        target = max(1, int(n * keep))
        st, vo, fo, cid = ctx.picasso_decimate(v, f, target, **over)
        ref = oracle.decimate(V, F, target)
        if drop:
            ref = oracle.drop_unreferenced(ref)
        np.testing.assert_array_equal(cid.cpu().numpy(), ref["cluster_id"])
        np.testing.assert_array_equal(fo.cpu().numpy(), ref["facets"])
        np.testing.assert_array_equal(vo.cpu().numpy().view(np.uint32), ref["verts"].view(np.uint32))
