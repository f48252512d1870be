"""A context tuned on a large batch, at a small one (GPU)."""
import numpy as np
import pytest

from gpu_util import say
from paper_1008_1371_amd import workloads as W

pytestmark = pytest.mark.gpu

CACHE = ('{"entries": [\n  {"batched_bucket": 3, "threads": 256, "problems_class": 4},'
         '\n  {"batched_schedule": 0, "mode": 0, "problems_class": 4}\n]}\n')


# 16 problems of order 250 to 256 take 20 ms at what wins for thousands (the
# persistent launch, 256 threads) and 4.6 in grouped launches.
def test_small_batch_keeps_its_speed(tmp_path, monkeypatch):
    import torch

    from paper_1008_1371_amd import hsvd as H
    cache = tmp_path / "tune.json"
    cache.write_text(CACHE)
    monkeypatch.setenv("HSVD_AUTOTUNE_CACHE", str(cache))
    ns = [250 + k % 7 for k in range(16)]
    flat, offs = W.pack_batch([W.gaussian(n, seed=k) for k, n in enumerate(ns)])
    voffs = np.concatenate([[0], np.cumsum(ns)[:-1]]).astype(np.int64)
    G = torch.from_numpy(flat).cuda()
    with H.Context(0) as ctx:
        ms = {}
        for mode in (2, 1):
            R = [H.hsvd_solve_batched(ctx, ns, [n // 2 for n in ns], G, offs, voffs, H.hsvd_default_params(batch_mode=mode))
                 for _ in range(4)]
            ms[mode] = min(r["infos"][0]["ms_total"] for r in R)
        say("default", ms[2], "grouped", ms[1])
        assert ms[2] <= 1.6 * ms[1]
        # tuning at this size adds its own entries and keeps the others
        H.hsvd_autotune_batched(ctx, ns, [n // 2 for n in ns])
        text = cache.read_text()
        assert '"batched_bucket": 3, "threads": 256, "problems_class": 4}' in text
        assert '"batched_schedule": 0, "mode": 0, "problems_class": 4}' in text
        assert text.count('"problems_class": 0}') == 3  # a width, a schedule per precision
        assert H.hsvd_batched_schedule(ctx, H.FP64) in (0, 1)
