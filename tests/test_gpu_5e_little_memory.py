"""Solves when the device has little memory left (GPU).  In batches what speed
alone asks for -- groups of launches side by side, many resident workgroups --
gives way, and the results are those of a context with all the memory."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

GIB = 1 << 30


class Held:
    """All device memory but `keep` bytes.  Taken until no 64 MiB are left, as
    the runtime gives up memory of its own (the kernels' private memory) when
    an allocation would fail, and does not report it as free before."""

    def __init__(self, keep):
        import torch
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        kept = torch.empty(keep, dtype=torch.uint8, device="cuda:0")
        self.blocks = []
        size = 32 * GIB
        while size >= 64 << 20:
            try:
                self.blocks.append(torch.empty(size, dtype=torch.uint8, device="cuda:0"))
            except torch.cuda.OutOfMemoryError:
                size //= 2
        del kept
        torch.cuda.empty_cache()

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        import torch
        self.blocks.clear()
        torch.cuda.empty_cache()


# 900 MB of workspace are asked for; what follows is this thread's next kernel,
# torch's, and the library's next solve.
def test_out_of_memory_leaves_no_error_behind():
    import torch

    from paper_1008_1371_amd import hsvd as H
    n = 4096
    G = torch.randn((n, n), dtype=torch.float64, device="cuda:0")
    g = torch.eye(100, dtype=torch.float64, device="cuda:0") * 2.0
    out = {k: torch.empty((n, n), dtype=torch.float64, device="cuda:0").t() for k in ("U", "V")}
    with H.Context(0) as ctx:
        with Held(GIB // 2):
            say("left", torch.cuda.mem_get_info()[0] / GIB, "GiB")
            R = H.hsvd_solve(ctx, G, n // 2, H.hsvd_default_params(precision=H.MIXED), out=out, check=False)
            assert R["status"] == H.E_NOMEM
            S = H.hsvd_solve(ctx, g, 50, H.hsvd_default_params(algo=H.BLOCK), check=False)
            assert S["status"] == 0 and bool((S["sigma"] == 2.0).all())


def _batch(ns):
    import torch
    sizes = np.asarray(ns, dtype=np.int64) ** 2
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    voffs = np.concatenate([[0], np.cumsum(ns)[:-1]]).astype(np.int64)
    gen = torch.Generator(device="cuda:0").manual_seed(len(ns))
    G = torch.randn(int(sizes.sum()), dtype=torch.float64, device="cuda:0", generator=gen)
    return G, offs, voffs


# The whole batch asks for 2.2 GiB (7 groups of 11 mixed problems; the largest
# alone 0.5) and 2.7 GiB (1024 workgroups' slots of mixed problems).
@pytest.mark.parametrize("ns,mode,keep", [([640 + 64 * (k % 7) for k in range(77)], 1, 1.6),
                                          ([8 + k % 5 for k in range(2000)], 0, 2.2)])
def test_batch_fits_what_is_left(ns, mode, keep):
    import torch

    from paper_1008_1371_amd import hsvd as H
    G, offs, voffs = _batch(ns)
    prm = H.hsvd_default_params(precision=H.MIXED, batch_mode=mode)
    args = (ns, [n // 3 for n in ns], G, offs, voffs, prm)
    with H.Context(0) as ctx:
        ref = H.hsvd_solve_batched(ctx, *args, check=False)
    out = {"sigma": torch.empty_like(ref["sigma"]), "U": torch.empty_like(G), "V": torch.empty_like(G),
           "lambda": torch.empty_like(ref["lam"])}
    with H.Context(0) as ctx, Held(int(keep * GIB)):
        say("left", torch.cuda.mem_get_info()[0] / GIB, "GiB")
        R = H.hsvd_solve_batched(ctx, *args, out=out, check=False)
    assert ref["status"] == 0 and R["status"] == 0
    for k in ("sigma", "lam", "U", "V"):
        assert torch.equal(R[k], ref[k]), k
