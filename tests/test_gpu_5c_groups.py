"""Groups of a batch side by side (GPU): the results of a batch of many orders
are those of each order's problems on their own."""
import numpy as np
import pytest

from gpu_util import say
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run(ctx, ns, Gs, **prm):
    import torch

    from paper_1008_1371_amd import hsvd as H
    flat, offs = W.pack_batch(Gs)
    voffs = np.concatenate([[0], np.cumsum(ns)[:-1]]).astype(np.int64)
    return H.hsvd_solve_batched(ctx, ns, [n // 3 for n in ns], torch.from_numpy(flat).cuda(), offs, voffs,
                                H.hsvd_default_params(**prm), check=False), offs, voffs


# One group alone, several at once, more block pairs than run at once (4 per
# compute unit, 256 of them: 700 problems of one pair, 300 of two, the rest),
# as graphs and as stream launches.  A problem's mixed trajectory depends on
# its group's sweeps only.
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("orders,graph", [([300], 1), ([300], 0), ([40, 100, 180, 250, 310, 390, 450], 1),
                                          ([40, 100, 180, 250, 310, 390, 450], 0),
                                          ([33] * 700 + [65] * 300 + [130, 257, 700], 1)])
def test_groups_side_by_side(hsvd_ctx, orders, precision, graph):
    import torch
    say("groups", len(orders), precision, graph)
    Gs = [W.gaussian(n, seed=k) for k, n in enumerate(orders)]
    prm = dict(precision=precision, graph=graph, batch_mode=1)
    R, offs, voffs = _run(hsvd_ctx, orders, Gs, **prm)
    assert R["status"] == 0
    for r in sorted({(n + 63) // 64 for n in orders}):
        ids = [k for k, n in enumerate(orders) if (n + 63) // 64 == r]
        S, o, v = _run(hsvd_ctx, [orders[k] for k in ids], [Gs[k] for k in ids], **prm)
        for z, k in enumerate(ids):
            n = orders[k]
            for key, at, own, size in (("sigma", voffs, v, n), ("lam", voffs, v, n), ("U", offs, o, n * n), ("V", offs, o, n * n)):
                a, b = R[key][at[k]:at[k] + size], S[key][own[z]:own[z] + size]
                assert torch.equal(a, b), (key, n)
            for key in ("status", "sweeps", "sweeps_fp32", "rotations", "skips", "reorth_iters", "code"):
                assert R["infos"][k][key] == S["infos"][z][key], (key, n)


# Before tuning few FP64 problems take the grouped launches; both schedules
# give the same bits, so the default does too.
@pytest.mark.parametrize("count", [1, 128, 129, 330])
def test_default_schedule(hsvd_ctx, count):
    import torch
    orders = [8 + (37 * k) % (120 if count in (128, 129) else 249) for k in range(count)]
    say("default schedule", count)
    Gs = [W.gaussian(n, seed=k) for k, n in enumerate(orders)]
    R = [_run(hsvd_ctx, orders, Gs, batch_mode=mode)[0] for mode in (2, 0, 1)]
    for other in R[1:]:
        for key in ("sigma", "lam", "U", "V"):
            assert torch.equal(R[0][key], other[key]), key
