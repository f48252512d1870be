"""Batches of orders far below a block pair's 64 columns (GPU): most inner steps
rotate nothing, and the 256-thread circle solve then only moves its entries."""
import numpy as np
import pytest

from gpu_util import say
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


# The persistent launch takes the 256-thread form, the grouped launches of at
# most 512 block pairs the 1024-thread one, which turns every block in every
# step: the results have to be equal bit for bit.  Diagonal and integer inputs
# bring exact and negative zeros.
@pytest.mark.parametrize("kind", ["gauss", "diagonal", "integer"])
@pytest.mark.parametrize("ordering,sort", [(0, 1), (1, 1), (0, 0)])
def test_tiny_orders_both_forms(hsvd_ctx, ordering, sort, kind):
    import torch

    from paper_1008_1371_amd import hsvd as H
    ns = [1, 2, 3, 5, 8, 13, 21, 34, 55, 64] * 12
    say("tiny orders", ordering, sort, kind)
    Gs = []
    for k, n in enumerate(ns):
        G = W.gaussian(n, seed=600 + k)
        if kind == "diagonal":
            G = np.diag(np.diag(G)) * np.where(G < 0.0, -1.0, 1.0)
        elif kind == "integer":
            G = np.triu(np.rint(2.0 * G), 1) - np.diag(np.arange(1.0, n + 1.0))
        Gs.append(G)
    flat, offs = W.pack_batch(Gs)
    voffs = np.concatenate([[0], np.cumsum(ns)[:-1]]).astype(np.int64)
    Gd = torch.from_numpy(flat).cuda()
    R = [H.hsvd_solve_batched(hsvd_ctx, ns, [n // 2 for n in ns], Gd, offs, voffs,
                              H.hsvd_default_params(ordering=ordering, sort=sort, batch_mode=mode, max_sweeps=30),
                              check=False) for mode in (0, 1)]
    assert R[0]["status"] == R[1]["status"] and np.array_equal(R[0]["statuses"], R[1]["statuses"])
    if kind != "integer":
        assert R[0]["status"] == 0
    for k in ("sigma", "lam", "U", "V"):
        a, b = R[0][k].view(torch.int64), R[1][k].view(torch.int64)
        assert torch.equal(a, b), k
    for k in ("sweeps", "rotations", "skips", "active_pairs", "code"):
        assert [i[k] for i in R[0]["infos"]] == [i[k] for i in R[1]["infos"]], k
