"""Batches on a stream of the caller's own (GPU): the groups that run side by
side start after what is queued there, and what is queued there next comes
after them."""
import numpy as np
import pytest

from gpu_util import say
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


# Six groups side by side, alone and beside a persistent launch.  The inputs
# are the last link of a chain of products still running when the call is
# made, the outputs are overwritten right after it; both on the same stream.
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("mode,graph", [(1, 1), (1, 0), (0, 1)])
def test_groups_keep_stream_order(mode, graph, precision):
    import torch

    from paper_1008_1371_amd import hsvd as H
    ns = [40, 100, 180, 250, 310, 390] * 2
    say("caller's stream", mode, graph, precision)
    flat, offs = W.pack_batch([W.gaussian(n, seed=k) for k, n in enumerate(ns)])
    voffs = np.concatenate([[0], np.cumsum(ns)[:-1]]).astype(np.int64)
    ps = [n // 3 for n in ns]
    prm = H.hsvd_default_params(precision=precision, graph=graph, batch_mode=mode)
    G = torch.from_numpy(flat).cuda()
    with H.Context(0) as ctx:
        ref = H.hsvd_solve_batched(ctx, ns, ps, G, offs, voffs, prm)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream), H.Context(0) as ctx:
        out = {"sigma": torch.zeros_like(ref["sigma"]), "U": torch.zeros_like(G), "V": torch.zeros_like(G),
               "lambda": torch.zeros_like(ref["lam"])}
        A = torch.eye(4096, dtype=torch.float64, device="cuda:0")
        late = torch.zeros_like(G)
        for _ in range(20):
            A = A @ A
        late.copy_(G * A[0, 0])
        H.hsvd_solve_batched(ctx, ns, ps, late, offs, voffs, prm, out=out)
        got = {k: v.clone() for k, v in out.items()}
        late.zero_()
        for v in out.values():
            v.zero_()
        stream.synchronize()
    for key, k in (("sigma", "sigma"), ("U", "U"), ("V", "V"), ("lambda", "lam")):
        assert torch.equal(got[key], ref[k]), key
