"""Cross inner solve of the block path (GPU): sign patterns of the block pairs,
and entries outside the range of the short rotation form."""
import numpy as np
import pytest

import pins
from gpu_util import run_lib, say
from parity import compare, twin_spread
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


# p = 0 and n: every pair trigonometric; 64: blocks of one sign, trigonometric
# and hyperbolic pairs of blocks; 33 and 95: a block with columns of both signs.
# Scales 2^-245 and 2^245: squared norms beyond 2^-480 and 2^480, where the
# pairs take the exact rotation form.
@pytest.mark.parametrize("scale", [0, -245, 245])
@pytest.mark.parametrize("n,p", [(128, 0), (128, 128), (128, 64), (128, 33), (97, 95), (190, 64)])
def test_cross_sign_patterns(hsvd_ctx, n, p, scale):
    G = np.ldexp(W.gaussian(n, seed=700 + n + p), scale)
    say("cross", n, p, scale)
    spread, ref = twin_spread(G, p, block=32)
    gate = max(1e-12, 10 * max(spread["U"], spread.get("V", 0.0)))
    res = run_lib(hsvd_ctx, G, p, algo=2)
    e = compare(res, ref, p)
    assert res["status"] == 0 and e["sigma_norm"] <= 1e-12 and e["U"] <= gate and e["V"] <= gate, (e, spread)
    if scale == 0:
        pins.check_invariants(G, p, res, tol=ref["tol"])
