"""GPU parity of kvsched_sortedF with the CPU oracle where its variants meet: sizes around the one-workgroup
variants' tiles and around the runs of the many-workgroup one, keys that do not fit in 64 bits, completion times
beyond the profile test's buckets, batches on either side of what one wavefront decides."""
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


def _lengths(rng, kind, n):
    if kind == "tiny":
        return rng.integers(1, 9, n), rng.integers(1, 9, n)
    if kind == "same":
        return np.full(n, 3), np.full(n, 5)
    if kind == "bimodal":
        return np.where(rng.random(n) < 0.5, 1, 4096), np.where(rng.random(n) < 0.5, 4096, 1)
    if kind == "huge":  # decode lengths far beyond any bucket table
        return rng.integers(1, 1 << 20, n), rng.integers(1, 1 << 22, n)
    return np.clip(rng.lognormal(4.8, 0.8, n), 4, 2048), np.clip(rng.lognormal(5.3, 0.9, n), 1, 2048)


def _check(ctx, s, o, M, feas, tie):
    import torch

    print(f"sortedF sizes: n={len(s)} M={M} feas={feas} tie={tie}", flush=True)
    order_o, ends_o, F_o = oracle.sortedF(s, o, M, tie, feas)
    order, ends, F, nb = ctx.sortedF(torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0"), M, tie, feas)
    k = int(nb.item())
    assert ctx.device_status() == 0
    assert k == len(ends_o) and (ends.cpu().numpy()[:k] == ends_o).all()
    assert (order.cpu().numpy() == order_o).all()
    assert np.allclose(F.cpu().numpy()[:k], F_o, rtol=1e-12, atol=0.0)
    assert (ends.cpu().numpy()[k:] == 0).all() and (F.cpu().numpy()[k:] == 0).all()


@pytest.mark.parametrize("feas", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 6143, 17000])
def test_sizes_around_the_tiles(ctx, n, feas):
    rng = np.random.default_rng(n)
    for kind, per in (("chat", 60), ("chat", 4), ("tiny", 5), ("bimodal", 25), ("same", 3)):
        s, o = (x.astype(np.int32) for x in _lengths(rng, kind, n))
        M = max(int((s.astype(np.int64) + o).max()), int(per * n))
        _check(ctx, s, o, M, feas, n & 1)


@pytest.mark.parametrize("feas", [0, 1])
@pytest.mark.parametrize("n", [50, 700, 2000, 3000, 5000])
def test_keys_and_times_that_do_not_fit(ctx, n, feas):
    rng = np.random.default_rng(n)
    s, o = (x.astype(np.int32) for x in _lengths(rng, "huge", n))
    for M in ((1 << 30) - 1, 3 * int((s.astype(np.int64) + o).max())):
        _check(ctx, s, o, M, feas, 0)


@pytest.mark.parametrize("feas", [0, 1])
def test_batches_around_one_wavefronts_reach(ctx, feas):
    for n in (3000, 9000):
        for K in (62, 64, 66, 254, 255, 256, 257, 258, 600):
            s, o = np.full(n, 2, dtype=np.int32), np.full(n, 2, dtype=np.int32)
            _check(ctx, s, o, 4 * K, feas, K & 1)


def test_extents_around_what_is_found_for_all_places(ctx):
    n = 9000
    for K in (2046, 2047, 2048, 2049, 2300):
        s, o = np.full(n, 2, dtype=np.int32), np.full(n, 2, dtype=np.int32)
        o[K // 2 :: K] = 900  # (batches shorter than their extents)
        for M in (4 * K + 1000, 4 * K + 1002):
            _check(ctx, s, o, M, 0, K & 1)


@pytest.mark.parametrize("feas", [0, 1])
def test_chains_longer_than_the_part_held_in_lds(ctx, feas):
    rng = np.random.default_rng(feas)
    for n in (40959, 40961, 73727, 73729, 150000):
        s, o = rng.integers(1, 9, n).astype(np.int32), rng.integers(1, 9, n).astype(np.int32)
        o[rng.integers(0, n, 20)] = 3000
        _check(ctx, s, o, 60000, feas, n & 1)  # (a few extents that are not found for all places among many that are)
        _check(ctx, s, o, 3100, feas, n & 1)


@pytest.mark.parametrize("kind,per,n", [("bimodal", 60, 20000), ("chat", 8, 9000), ("chat", 75, 2049), ("chat", 79, 30000),
                                        ("tiny", 1, 5000), ("same", 1, 6000), ("mixed", 100, 12000), ("uniform", 300, 7000)])
def test_profile_extents_found_for_all_places(ctx, kind, per, n):
    """Completion times of one row, of 2048, 2049 and 4096; many requests that join where few leave; ties of both kinds."""
    rng = np.random.default_rng(n)
    if kind == "mixed":
        s, o = _lengths(rng, "chat", n)
        long = rng.random(n) < 0.3
        s, o = np.where(long, rng.integers(2048, 8193, n), s), np.where(long, rng.integers(100, 501, n), o)
    elif kind == "uniform":
        s, o = rng.integers(1, 1000, n), rng.integers(1, 4097, n)
    else:
        s, o = _lengths(rng, kind, n)
    s, o = s.astype(np.int32), o.astype(np.int32)
    M = max(int((s.astype(np.int64) + o).max()), int(per * n))
    for o_max in (int(o.max()), 2048, 2049, 4096, 4097):
        if o_max >= o.max() and o_max + s[5] <= M:
            o[5] = o_max
            _check(ctx, s, o, M, 1, n & 1)


def test_a_faulty_request_gives_no_batches(ctx):
    import torch

    for n in (40, 1500, 5000):
        s, o = np.full(n, 2, dtype=np.int32), np.full(n, 2, dtype=np.int32)
        o[n // 2] = 0
        for feas in (0, 1):
            _, ends, F, nb = ctx.sortedF(torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0"), 100, 0, feas)
            assert int(nb.item()) == 0 and ctx.device_status() & 1
            assert (ends == 0).all() and (F == 0).all()
