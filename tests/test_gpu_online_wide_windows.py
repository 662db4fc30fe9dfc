"""GPU parity of kvsched_online with the CPU oracle for windows beyond one row of registers: batches that stay in the lanes and
batches that do not, exchanges that come to reach beyond the first 64 requests, many requests of one decode length, and
the lanes of eight to sixty-four that take part in the exchanges."""
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


def _check(ctx, a, s, o, M, cases):
    import torch

    n = len(a)
    desc = np.array([[0, n, *c[:3], *c[3], k * n] for k, c in enumerate(cases)], dtype=np.int32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x.astype(np.int32))).to("cuda:0")
    comp, stats = ctx.online(dev(desc), dev(a), dev(s), dev(o), M,
                             torch.full((len(cases) * n,), -7, dtype=torch.int32, device="cuda:0"), backlog_cap=512)
    assert ctx.device_status() == 0
    for k, c in enumerate(cases):
        _, c_o, st_o = oracle.online(a, s, o, M, *c)
        assert tuple(int(x) for x in stats[k]) == st_o, c
        assert (comp[k * n : (k + 1) * n].cpu().numpy() == c_o).all(), c


@pytest.mark.parametrize("waiting", [7, 9, 31, 33, 66, 130, 200, 300])
@pytest.mark.parametrize("at_once", [2, 8, 30, 63, 64, 65, 90])
def test_batches_about_a_row(ctx, waiting, at_once):
    """Batches of about `at_once` requests of some 100 tokens, and half as many."""
    rng = np.random.default_rng(100 * waiting + at_once)
    n = waiting + 20
    a = np.concatenate([np.zeros(waiting), np.sort(rng.integers(0, 200, 20))]).astype(np.int32)
    o = rng.integers(1, 100, n).astype(np.int32)
    s = (rng.integers(90, 110, n) - o // 2).astype(np.int32)
    cases = [(3, 10, 300, (1, 2)), (3, 1, 300, (0, 1)), (3, 3, 129, (1, 4))]
    for part in (1, 2):
        M = max(160, 125 * at_once // part)
        print(f"online: {waiting} waiting, {at_once} at once, M={M}", flush=True)
        _check(ctx, a, s, o, M, cases)


@pytest.mark.parametrize("waiting", [64, 65, 150, 290])
def test_exchanges_that_reach_further(ctx, waiting):
    """Small requests of long decodes first: each exchange for a shorter one frees or takes tokens, so that the places within
    reach move; and requests of one decode length, of which none is exchanged."""
    rng = np.random.default_rng(waiting)
    n = waiting + 6
    a = np.zeros(n, dtype=np.int32)
    size = np.sort(rng.integers(60, 60 + n, n)).astype(np.int32)
    o = np.clip(59 - np.arange(n) // 6 + rng.integers(-3, 4, n), 1, 59).astype(np.int32)
    for M in (360, 2000, 62 * 64, 66 * 70, 100 * n):  # (the largest request has up to 355 tokens)
        print(f"online: reach, {waiting} waiting, M={M}", flush=True)
        _check(ctx, a, size - o, o, M, [(3, 10, 300, (1, 2)), (3, 1, 200, (0, 1))])
    o[:] = 40
    _check(ctx, a, size, o, 5000, [(3, 10, 300, (1, 2))])
