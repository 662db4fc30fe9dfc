"""Local Swap Search with two places a lane and next to it: backlogs of about 128 and 256 places that fit, batches that begin
at any place of a group of eight, members whose last one leaves, many requests of one size behind the last member."""
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


def _check(ctx, s, o, M):
    import torch

    print(f"local swap places: n={len(s)} M={M}", flush=True)
    want = oracle.local_swap(s, o, M, True)
    order, ends, F, swaps, nb = ctx.local_swap(torch.from_numpy(s).cuda(), torch.from_numpy(o).cuda(), M)
    k = int(nb.item())
    assert k == len(want[1]) and ctx.device_status() == 0
    assert (order.cpu().numpy() == want[0]).all()
    assert (ends.cpu().numpy()[:k] == want[1]).all()
    assert (swaps.cpu().numpy()[:k] == want[3]).all()
    assert np.allclose(F.cpu().numpy()[:k], want[2], rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 126, 127, 128, 129, 130, 135, 255, 256, 257, 300])
def test_about_two_places_a_lane(ctx, n):
    rng = np.random.default_rng(n)
    for per in (3, 11, 60, n):  # requests a batch, about
        s, o = rng.integers(1, 40, n).astype(np.int32), rng.integers(1, 400, n).astype(np.int32)
        _check(ctx, s, o, max(int((s + o).max()), int(per * (s + o).mean())))


@pytest.mark.parametrize("n", [100, 300, 1500])
def test_requests_of_one_size(ctx, n):
    rng = np.random.default_rng(n)
    s, o = np.where(rng.random(n) < 0.5, 1, 400).astype(np.int32), np.where(rng.random(n) < 0.5, 400, 1).astype(np.int32)
    for M in (801, 2500, 30 * n, 200 * n):
        _check(ctx, s, o, max(M, 801))
    total = rng.integers(60, 64, n).astype(np.int32)  # (four sizes, the decode lengths free)
    o = rng.integers(1, 60, n).astype(np.int32)
    for M in (70, 700, 20 * n):
        _check(ctx, total - o, o, max(M, 64))
