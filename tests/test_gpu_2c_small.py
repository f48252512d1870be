"""One-workgroup pairwise solves (r <= 128, GPU): the row and slot layouts at
their edges, bit-identical to the per-step visits of the persistent kernel."""
import numpy as np
import pytest

from gpu_util import run_lib, say
from parity import compare, twin_spread
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


# rows per wave change at 16, 32 and 64, slots that divide a wave (powers of
# two) rotate it whole; scales 2^-245 and 2^245 take the general rotation
# routine
@pytest.mark.parametrize("want_v", [1, 0])
@pytest.mark.parametrize("n,p,scale", [(2, 2, 0), (15, 7, 0), (16, 0, 0), (17, 17, 0), (18, 9, 0), (32, 11, 0),
                                       (33, 20, 0), (34, 34, 0), (63, 31, 0), (64, 40, -245), (65, 1, 0), (90, 45, 245),
                                       (127, 60, 0), (128, 128, 0), (128, 64, -245)])
def test_small_matches_steps(hsvd_ctx, n, p, scale, want_v):
    G = np.ldexp(W.gaussian(n, seed=900 + n), scale)
    say("small", n, p, scale, want_v)
    a = run_lib(hsvd_ctx, G, p, algo=1, want_v=want_v)
    b = run_lib(hsvd_ctx, G, p, algo=1, want_v=want_v, persistent=2)
    for k in ("status", "sweeps"):
        assert a[k] == b[k], k
    for k in ("code", "rotations", "skips", "max_t_last"):
        assert a["info"][k] == b["info"][k], k
    for k in ("sigma", "U", "V", "lam", "perm"):
        assert (a[k] is None and b[k] is None) or np.array_equal(a[k], b[k]), k
    spread, ref = twin_spread(G, p)
    e = compare(a, ref, p)
    assert a["status"] == 0 and e["sigma_norm"] <= 1e-12 and e["U"] <= max(1e-12, 10 * spread["U"]), (e, spread)


@pytest.mark.parametrize("max_sweeps,sort", [(1, 1), (2, 0)])
def test_small_stops_early(hsvd_ctx, max_sweeps, sort):
    G = W.gaussian(70, seed=970)
    a = run_lib(hsvd_ctx, G, 30, algo=1, max_sweeps=max_sweeps, sort=sort)
    b = run_lib(hsvd_ctx, G, 30, algo=1, max_sweeps=max_sweeps, sort=sort, persistent=2)
    assert a["status"] == b["status"] == -2 and a["sweeps"] == max_sweeps
    for k in ("sigma", "U", "V", "lam", "perm"):
        assert np.array_equal(a[k], b[k]), k
    assert np.all(np.isfinite(a["sigma"]))
