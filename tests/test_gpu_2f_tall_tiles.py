"""Pairwise tiles of the tallest class of columns, 1537 to 2048 rows (GPU; the
seven classes below are test_gpu_2d_tiles.py's), and the step launches that a
fixed scratch without room for the tiles falls back to."""
import pytest

from gpu_util import say, to_dev
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


def _equal(a, b):
    import torch
    for k in ("sigma", "lam", "U", "V", "perm"):
        assert (a[k] is None and b[k] is None) or torch.equal(a[k], b[k]), k
    for k in ("status", "sweeps", "rotations", "skips", "steps", "code", "max_t_last"):
        assert a["info"][k] == b["info"][k], k


# the first order of the class, a ragged one (its last run holds three
# positions of four), the last order that goes in tiles
@pytest.mark.parametrize("want_v", [1, 0])
@pytest.mark.parametrize("n,p", [(1537, 700), (1990, 1990), (2048, 1024)])
def test_tall_tiles_equal_steps(hsvd_ctx, n, p, want_v):
    from paper_1008_1371_amd import hsvd as H
    say("tall tiles", n, p, want_v)
    G = to_dev(W.gaussian(n, seed=970 + n))
    R = [H.hsvd_solve(hsvd_ctx, G, p, H.hsvd_default_params(algo=H.PAIRWISE, persistent=k, max_sweeps=2, want_v=want_v),
                      check=False) for k in (0, 1)]
    assert R[0]["info"]["kernel_launches"][0] < R[0]["info"]["steps"]
    _equal(R[0], R[1])


# With V the scratch array has room for the tiles' rotations up to bordered
# order 2040, and for a solve without them up to 2044.
@pytest.mark.parametrize("n,tiles", [(2039, True), (2040, True), (2041, False), (2044, False)])
def test_fixed_scratch_without_tiles(hsvd_ctx, n, tiles):
    from paper_1008_1371_amd import hsvd as H
    say("fixed scratch", n, tiles)
    G = to_dev(W.gaussian(n, seed=970 + n))
    prm = H.hsvd_default_params(algo=H.PAIRWISE, max_sweeps=1)
    a = H.hsvd_solve(hsvd_ctx, G, 900, prm, check=False)
    b = H.hsvd_solve_noalloc(hsvd_ctx, G, 900, prm, check=False)
    launches, steps = b["info"]["kernel_launches"][0], b["info"]["steps"]
    assert launches < steps if tiles else launches == steps == n + n % 2
    _equal(a, b)


def test_fixed_scratch_largest_pairwise_order(hsvd_ctx):
    from paper_1008_1371_amd import hsvd as H
    R = H.hsvd_solve_noalloc(hsvd_ctx, to_dev(W.gaussian(2045, seed=1)), 900, H.hsvd_default_params(algo=H.PAIRWISE),
                             check=False)
    assert R["status"] == H.E_SIZE
