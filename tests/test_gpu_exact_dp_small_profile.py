"""GPU parity with the CPU oracle of exact batches under the profile constraint where the tables fit one workgroup's LDS: the
largest budgets, batch sizes and decode lengths of that kernel, in whose test at a completion (load + o k <= M) they meet."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M,s_max,o_max", [(1, 8191, 1, 8190), (6, 4095, 1500, 2400), (40, 2047, 300, 1500), (64, 255, 9, 230), (150, 127, 2, 120),
                                             (200, 63, 1, 60), (300, 64, 3, 3)])
@pytest.mark.parametrize("tie", [0, 1])
def test_profile(n, M, s_max, o_max, tie):
    from paper_2508_06133_amd import kvsched
    import torch

    rng = np.random.default_rng(n + M)
    s = rng.integers(1, s_max + 1, n).astype(np.int32)
    o = np.where(rng.random(n) < 0.7, rng.integers(1, 1 + max(1, o_max // 16), n), rng.integers(1, o_max + 1, n)).astype(np.int32)
    o = np.minimum(o, M - s)
    print(f"exact_dp, small tables, profile: n={n} M={M} tie={tie}", flush=True)
    order_o, ends_o, F_o = oracle.exact_phase1(s, o, M, 1, tie)
    ctx = kvsched.Context(0)
    try:
        order, ends, F, nb = ctx.exact_dp(torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0"), M, 1, tie)
        k = int(nb.item())
        assert ctx.device_status() == 0 and k == len(ends_o)
        assert (ends.cpu().numpy()[:k] == ends_o).all() and (order.cpu().numpy() == order_o).all()
        assert np.allclose(F.cpu().numpy()[:k], F_o, rtol=1e-12, atol=0.0)
    finally:
        ctx.close()
