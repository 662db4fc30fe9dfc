"""GPU parity of exact batches with the CPU oracle in the one-workgroup kernel, which offers two requests a step: one request and odd
numbers, rows of one part of 64 loads and of more parts than there are wavefronts, batches of one request, equal lengths."""
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


def _check(ctx, s, o, M, feas, tie):
    import torch

    print(f"exact_dp, small tables: n={len(s)} M={M} feas={feas} tie={tie}", flush=True)
    order_o, ends_o, F_o = oracle.exact_phase1(s, o, M, feas, tie)
    order, ends, F, nb = ctx.exact_dp(torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0"), M, feas, tie)
    k = int(nb.item())
    assert ctx.device_status() == 0 and k == len(ends_o)
    assert (ends.cpu().numpy()[:k] == ends_o).all() and (order.cpu().numpy() == order_o).all()
    assert np.allclose(F.cpu().numpy()[:k], F_o, rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("feas", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 16, 17, 33])
@pytest.mark.parametrize("M", [2, 62, 63, 64, 65, 127, 128, 129, 191, 192])
def test_numbers_of_requests_and_loads(ctx, n, M, feas):
    rng = np.random.default_rng(100 * n + M)
    for most in (2, 9, M):
        s = rng.integers(1, max(2, min(most, M) // 2 + 1), n).astype(np.int32)
        o = np.minimum(rng.integers(1, max(2, min(most, M)), n), M - s).astype(np.int32)
        _check(ctx, s, o, M, feas, n & 1)
    _check(ctx, np.full(n, 1, np.int32), np.full(n, 1, np.int32), M, feas, 1)


@pytest.mark.parametrize("feas", [0, 1])
@pytest.mark.parametrize("n,M,least", [(7, 1023, 120), (5, 1024, 400), (9, 2047, 500), (4, 2500, 1300), (3, 4095, 2100)])
def test_long_rows(ctx, n, M, least, feas):
    """Few large requests: rows of up to 64 parts, which sixteen wavefronts step through."""
    rng = np.random.default_rng(n + M)
    s = rng.integers(least, least + least // 4, n).astype(np.int32)
    o = np.minimum(rng.integers(1, least // 2, n), M - s).astype(np.int32)
    for tie in (0, 1):
        _check(ctx, s, o, M, feas, tie)
