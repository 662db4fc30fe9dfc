"""GPU parity of kvsched_exact_dp with the CPU oracle where batches are decided without a table: numbers of requests around
the 256 that this takes, from no undecided request to more than can be tried (equal and nearly equal requests), sets of
equal metric, load and size in number, and the G metric."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2508_06133_amd import kvsched

    c = kvsched.Context(0)
    yield c
    c.close()


def _lengths(kind, n, M, rng):
    if kind == "chat":
        s, o = rng.lognormal(np.log(128), 0.8, n), rng.lognormal(np.log(200), 0.9, n)
    elif kind == "equal":  # one request n times over: the earliest ones make a batch
        s, o = np.full(n, M // 9), np.full(n, 17)
    elif kind == "few":  # equal sums of different requests
        s, o = 64 * rng.integers(1, 5, n), 64 * rng.integers(1, 5, n)
    elif kind == "near":  # one trade of value for load: every set of a size is within a few of the others
        o = rng.integers(400, 440, n)
        s = 3000 - 2 * o + rng.integers(0, 3, n)
    elif kind == "large":  # no more than two of them fit
        s, o = rng.integers(M // 4, M // 2, n), rng.integers(1, M // 2, n)
    s, o = np.clip(np.rint(s), 1, M - 1).astype(np.int32), np.rint(o).astype(np.int32)
    return s, np.clip(o, 1, M - s).astype(np.int32)


@pytest.mark.parametrize("kind,n,M", [("chat", 60, 8200), ("chat", 255, 9001), ("chat", 256, 8192), ("chat", 257, 9000), ("chat", 300, 8448),
                                      ("equal", 40, 9000), ("few", 64, 8192), ("few", 256, 8300), ("near", 50, 8500),
                                      ("near", 257, 8500), ("large", 100, 9000), ("large", 256, 60000)])
@pytest.mark.parametrize("alpha", [(0, 1), (2, 3)])
def test_batches(ctx, kind, n, M, alpha):
    from paper_2508_06133_amd import kvsched
    import torch

    s, o = _lengths(kind, n, M, np.random.default_rng(n + M))
    ds, do = torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0")
    for tie in (0, 1):
        print(f"exact_dp without tables: {kind} n={n} M={M} alpha={alpha} tie={tie}", flush=True)
        if alpha[0]:
            order_o, ends_o, F_o = oracle.exact_phase1(s, o, M, 0, tie, alpha)
            order, ends, F, _, nb = ctx.phase1_G(kvsched.SOLVER_EXACT_DP, ds, do, M, alpha, tie, 0)
        else:
            order_o, ends_o, F_o = oracle.exact_phase1(s, o, M, 0, tie)
            order, ends, F, nb = ctx.exact_dp(ds, do, M, 0, tie)
        k = int(nb.item())
        assert ctx.device_status() == 0 and k == len(ends_o)
        assert (ends.cpu().numpy()[:k] == ends_o).all() and (order.cpu().numpy() == order_o).all()
        assert np.allclose(F.cpu().numpy()[:k], F_o, rtol=1e-12, atol=0.0)
