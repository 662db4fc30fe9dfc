"""GPU parity of kvsched_sortedF with the CPU oracle where the many launches of a large construction change: places by
counting in groups of 32 and of 64, by sorted runs beyond; prefix sums with and without sums ahead; orders within batches of one
request, of thousands and across the 64 places of a workgroup; the length scan that the first launch makes."""
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

    s, o = np.asarray(s, dtype=np.int32), np.asarray(o, dtype=np.int32)
    print(f"sortedF counted places: n={len(s)} M={M} feas={feas} tie={tie}", flush=True)
    order_o, ends_o, F_o = oracle.sortedF(s, o, M, tie, feas)
    order, ends, F, nb = ctx.sortedF(torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0"), M, tie, feas)
    k = int(nb.item())
    assert ctx.device_status() == 0
    assert k == len(ends_o) and (ends.cpu().numpy()[:k] == ends_o).all()
    assert (order.cpu().numpy() == order_o).all()
    assert np.allclose(F.cpu().numpy()[:k], F_o, rtol=1e-12, atol=0.0)


def _chat(rng, n):
    return np.clip(rng.lognormal(4.8, 0.8, n), 4, 2048).astype(int), np.clip(rng.lognormal(5.3, 0.9, n), 1, 2048).astype(int)


@pytest.mark.parametrize("feas", [0, 1])
@pytest.mark.parametrize("n", [127, 128, 129, 1087, 8191, 8192, 8193, 12287, 12288, 12289, 16384, 16385])
def test_sizes(ctx, n, feas):
    rng = np.random.default_rng(n)
    s, o = _chat(rng, n)
    for per in (5, 60, 500):
        _check(ctx, s, o, max(4200, per * n), feas, n & 1)
    _check(ctx, s, o, (1 << 30) - 1, feas, 0)  # (keys hold ranks)
    o[n // 3] = 9000  # (completion times beyond the buckets)
    _check(ctx, s, o, max(12000, 60 * n), feas, 1)


@pytest.mark.parametrize("n", [1100, 9000])
def test_batches_across_the_places_of_a_workgroup(ctx, n):
    rng = np.random.default_rng(n)
    for K in (1, 2, 31, 63, 64, 65, 130, n):
        _check(ctx, np.full(n, 2), np.full(n, 2), 4 * K, 0, 1)
    o = rng.integers(1, 4, n)
    _check(ctx, rng.integers(1, 4, n), o, 6, 0, 0)   # (batches of one to three requests)
    _check(ctx, np.full(n, 1), rng.permutation(n) + 1, 1 << 29, 0, 1)  # (one batch, wide keys)


def test_a_faulty_request_and_a_good_call_after_it(ctx):
    import torch

    rng = np.random.default_rng(1)
    for n in (200, 1100, 9000, 13000, 40000):
        s, o = _chat(rng, n)
        for at, what in ((0, 0), (n - 1, -5), (n // 2, 1 << 29)):
            bad = o.copy()
            bad[at] = what
            for feas in (0, 1):
                _, ends, F, nb = ctx.sortedF(torch.from_numpy(s.astype(np.int32)).to("cuda:0"),
                                             torch.from_numpy(bad.astype(np.int32)).to("cuda:0"), 60 * n, 0, feas)
                assert int(nb.item()) == 0 and ctx.device_status() == 1
                assert (ends == 0).all() and (F == 0).all()
        _check(ctx, s, o, max(4200, 60 * n), 1, 0)


@pytest.mark.parametrize("n,omax", [(150, 2048), (1200, 2047), (1200, 255), (3000, 2049), (24000, 2048), (24000, 256)])
def test_extents_found_ahead_or_by_the_chain(ctx, n, omax):
    """One batch and more, extents around 16 and around 10000 requests, longest decodes around 2048 and full turns of 256 times."""
    rng = np.random.default_rng(n + omax)
    s, o = rng.integers(1, 400, n), rng.integers(1, omax + 1, n)
    o[: n // 8] = np.minimum(omax, 256 * rng.integers(1, 9, n // 8))
    o[n // 2] = omax
    total = int((s + o).sum())
    for M in (total, total - 1, total // 2, total // 7, 16 * total // n, 16 * total // n - 1, 10000 * total // n, 10000 * total // n + 1):
        _check(ctx, s, o, min(max(M, 400 + omax), (1 << 30) - 1), 1, n & 1)


@pytest.mark.parametrize("n,omax", [(129, 700), (200, 2048), (255, 2049), (256, 2048), (256, 9000), (257, 2048), (257, 5000)])
def test_no_extent_beyond_the_tests_of_one_wavefront(ctx, n, omax):
    """Up to 256 requests under the profile constraint, and one more: all in one batch, a few batches, one request each."""
    rng = np.random.default_rng(n + omax)
    s, o = rng.integers(1, 400, n), rng.integers(1, omax + 1, n)
    o[n // 2] = omax
    total = int((s + o).sum())
    for M in ((1 << 30) - 1, total, total - 1, total // 2, total // 3, total // 6, total // 20, 0):
        for tie in (0, 1):
            _check(ctx, s, o, max(M, 400 + omax), 1, tie)
