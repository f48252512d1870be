"""Circle inner solve (GPU): one block pair, both thread counts, sign patterns
and entries outside the range of the short rotation form."""
import numpy as np
import pytest

import pins
from gpu_util import run_lib, say
from parity import compare, twin_spread
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


def _run_batched(ctx, G, p):
    import torch

    from paper_1008_1371_amd import hsvd as H
    n = G.shape[0]
    zero = np.zeros(1, dtype=np.int64)
    R = H.hsvd_solve_batched(ctx, [n], [p], torch.from_numpy(G.ravel(order="F")).cuda(), zero, zero,
                             H.hsvd_default_params(), check=False)
    return dict(status=R["status"], sigma=R["sigma"].cpu().numpy(),
                U=R["U"].cpu().numpy().reshape(n, n, order="F"), V=R["V"].cpu().numpy().reshape(n, n, order="F"))


# p = 0 and 64: every pair trigonometric; 32: blocks of one sign each; 20 and
# 63: a block with columns of both signs; n = 41: a bordered pair.  Scales as
# in the cross solve's test: the exact rotation form.
@pytest.mark.parametrize("scale", [0, -245, 245])
@pytest.mark.parametrize("n,p", [(64, 0), (64, 64), (64, 32), (64, 20), (64, 63), (41, 13)])
def test_circle_sign_patterns(hsvd_ctx, n, p, scale):
    G = np.ldexp(W.gaussian(n, seed=900 + n + p), scale)
    say("circle", n, p, scale)
    spread, ref = twin_spread(G, p, block=32)
    gate = max(1e-12, 10 * max(spread["U"], spread.get("V", 0.0)))
    res = run_lib(hsvd_ctx, G, p, algo=2)
    for got in (res, _run_batched(hsvd_ctx, G, p)):
        e = compare(got, ref, p)
        assert got["status"] == 0 and e["sigma_norm"] <= 1e-12 and e["U"] <= gate and e["V"] <= gate, (e, spread)
    if scale == 0:
        pins.check_invariants(G, p, res, tol=ref["tol"])
