"""Solves when the device has little memory left (GPU)."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

GIB = 1 << 30


class Held:
    """All device memory but `keep` bytes, taken in blocks of at most 32 GiB."""

    def __init__(self, keep):
        import torch
        torch.cuda.empty_cache()
        self.blocks = []
        while True:
            free = torch.cuda.mem_get_info()[0]
            if free <= keep + (64 << 20):
                break
            try:
                self.blocks.append(torch.empty(min(free - keep, 32 * GIB), dtype=torch.uint8, device="cuda:0"))
            except torch.cuda.OutOfMemoryError:
                break

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
