"""Pairwise sweeps in tiles of 4 x 4 pairs (GPU): whole and ragged runs of
positions, every column height class, signs inside and between the runs."""
import numpy as np
import pytest

from gpu_util import say, to_dev
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


# r / 2 = 65 .. 68: runs of 4 with 1, 2, 3 and no positions in the last one;
# 193 .. 1025: the first order of each column height class, 1030: its twin
# with a ragged run.  The tiles see every pair's columns as the step-by-step
# order does, so the persistent kernel's results (the per-step arithmetic in
# that order) have to come out bit for bit.
@pytest.mark.parametrize("want_v", [1, 0])
@pytest.mark.parametrize("n,p", [(129, 129), (132, 0), (134, 67), (135, 30), (193, 100), (257, 20), (385, 384),
                                 (513, 256), (769, 301), (1025, 1000), (1030, 515)])
def test_tiles_equal_steps(hsvd_ctx, n, p, want_v):
    import torch

    from paper_1008_1371_amd import hsvd as H
    say("tiles", n, p, want_v)
    G = to_dev(W.gaussian(n, seed=970 + n))
    R = [H.hsvd_solve(hsvd_ctx, G, p, H.hsvd_default_params(algo=H.PAIRWISE, persistent=k, max_sweeps=3, want_v=want_v),
                      check=False) for k in (0, 1)]
    for k in ("sigma", "lam", "U", "V", "perm"):
        if R[0][k] is None:
            assert R[1][k] is None
            continue
        assert torch.equal(R[0][k], R[1][k]), k
    for k in ("status", "sweeps", "rotations", "skips", "steps", "code", "max_t_last"):
        assert R[0]["info"][k] == R[1]["info"][k], k
