"""Several host threads, each with a context and a stream of its own (GPU)."""
import threading

import numpy as np
import pytest

from gpu_util import say
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu


# Groups side by side (their sweeps captured as graphs while other threads
# allocate, launch and capture), the persistent launch, one workgroup, tiles
# and the block path, all at once: every result is that of the call alone.
def test_threads_do_not_disturb_each_other():
    import torch

    from paper_1008_1371_amd import hsvd as H
    ns = [40, 100, 180, 250, 310, 390]
    flat, offs = W.pack_batch([W.gaussian(n, seed=k) for k, n in enumerate(ns)])
    voffs = np.concatenate([[0], np.cumsum(ns)[:-1]]).astype(np.int64)
    G = torch.from_numpy(flat).cuda()
    single = {n: torch.from_numpy(np.asfortranarray(W.gaussian(n, seed=n))).cuda() for n in (90, 301, 520)}

    def batch(ctx, mode, precision):
        R = H.hsvd_solve_batched(ctx, ns, [n // 3 for n in ns], G, offs, voffs,
                                 H.hsvd_default_params(batch_mode=mode, precision=precision))
        return [R[k] for k in ("sigma", "lam", "U", "V")]

    def solve(ctx, n):
        R = H.hsvd_solve(ctx, single[n], n // 3)
        return [R[k] for k in ("sigma", "lam", "U", "V", "perm")]

    work = [lambda c: batch(c, 1, 0), lambda c: batch(c, 1, 1), lambda c: batch(c, 0, 1), lambda c: solve(c, 90),
            lambda c: solve(c, 301), lambda c: solve(c, 520)]
    with H.Context(0) as ctx:
        ref = [f(ctx) for f in work]
    torch.cuda.synchronize()
    wrong = []

    def run(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for rep in range(3):
                    with H.Context(0) as ctx:
                        for i in range(len(work)):
                            at = (i + k) % len(work)
                            got = work[at](ctx)
                            stream.synchronize()
                            if not all(torch.equal(a, b) for a, b in zip(got, ref[at])):
                                wrong.append((k, rep, at))
        except Exception as e:  # reported by the test's thread
            wrong.append((k, repr(e)))

    threads = [threading.Thread(target=run, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    say("threads", wrong)
    assert not wrong
