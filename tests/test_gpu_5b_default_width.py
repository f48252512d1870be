"""Width of the persistent batched launch before tuning (GPU): small batches
of every bucket of the largest order, whose workgroups hold more groups of
threads than a problem has block pairs, as many, or fewer."""
import numpy as np
import pytest

from gpu_util import say
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


# 1 to 4 block pairs per outer step (bordered orders 64 .. 256); the FP64
# results have to equal the grouped launches' bit for bit.
@pytest.mark.parametrize("ordering", [0, 1])
@pytest.mark.parametrize("ns", [[64], [65, 3], [128, 1, 64], [192], [129, 190, 70], [193], [256, 255, 150, 20]])
def test_default_width_equals_grouped(hsvd_ctx, ns, ordering):
    import torch

    from paper_1008_1371_amd import hsvd as H
    say("default width", ns, ordering)
    Gs = [W.gaussian(n, seed=950 + n) for n in ns]
    flat, offs = W.pack_batch(Gs)
    voffs = np.concatenate([[0], np.cumsum(ns)[:-1]]).astype(np.int64)
    Gd = torch.from_numpy(flat).cuda()
    R = [H.hsvd_solve_batched(hsvd_ctx, ns, [n // 3 for n in ns], Gd, offs, voffs,
                              H.hsvd_default_params(ordering=ordering, batch_mode=mode), check=False) for mode in (0, 1)]
    assert R[0]["status"] == 0 and R[1]["status"] == 0
    for k in ("sigma", "lam", "U", "V"):
        assert torch.equal(R[0][k], R[1][k]), k
    for k in ("sweeps", "rotations", "skips", "active_pairs", "code"):
        assert [i[k] for i in R[0]["infos"]] == [i[k] for i in R[1]["infos"]], k
