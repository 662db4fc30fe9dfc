"""The least latency where its halves decide: latencies beyond 32 bits that agree in either half, ties in other lanes, wavefronts and
workgroups, the largest latency, none at all."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 64, 65, 1024, 1025, 4096, 4097, 6145, 131073])
def test_wide_latencies(K):
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(K)
    ctx = kvsched.Context(0)
    try:
        for high, low in ((3, 3), (1, 2**32), (2**30, 2), (2**31, 2**32)):
            tel = (rng.integers(0, high, K).astype(np.int64) << 32) | rng.integers(0, low, K).astype(np.int64)
            tel[rng.random(K) < 0.4] = -1
            print(f"argmin: K={K} high={high} low={low}", flush=True)
            for alone in (None, int(rng.integers(K))):
                if alone is not None:  # (one valid entry, and the largest number there is)
                    tel[:] = -1
                    tel[alone] = np.iinfo(np.int64).max
                valid = np.flatnonzero(tel >= 0)
                want = (int(valid[np.argmin(tel[valid])]), int(tel[valid].min())) if len(valid) else (-1, -1)
                assert tuple(int(x) for x in ctx.argmin(torch.from_numpy(tel).to("cuda:0")).cpu().numpy()) == want
    finally:
        ctx.close()
