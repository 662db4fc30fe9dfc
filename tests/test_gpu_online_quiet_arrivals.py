"""GPU parity of kvsched_online with the CPU oracle where arrivals are waited for together: many requests arrive while the
head of the list waits for memory, the refresh comes with the growth of the backlog, after a period or never, and requests
of equal length leave the order within a batch to their ids."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _dev(x):
    import torch

    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def _run(a, s, o, M, policies, cap=512):
    import torch
    from paper_2508_06133_amd import kvsched

    n = len(a)
    desc = np.array([[0, n, *c[:3], *c[3], k * n] for k, c in enumerate(policies)], dtype=np.int32)
    ctx = kvsched.Context(0)
    try:
        comp, stats = ctx.online(_dev(desc), _dev(a), _dev(s), _dev(o), M,
                                 torch.full((len(policies) * n,), -7, dtype=torch.int32, device="cuda:0"), backlog_cap=cap)
        return comp.cpu().numpy(), stats.cpu().numpy(), ctx.device_status()
    finally:
        ctx.close()


RATIOS = [(1, 2), (3, 2), (7, 1), (0, 1), (1, 0), (1 << 19, 1 << 20), (1 << 30, 1)]


@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("rate", [0.2, 2.0, 30.0])
@pytest.mark.parametrize("period", [1, 7, 100000])
def test_arrivals_while_the_head_waits(equal, rate, period):
    rng = np.random.default_rng(int(10 * rate) + period)
    n = 200
    a = np.sort(rng.integers(0, int(n / rate) + 1, n)).astype(np.int32)
    s = rng.integers(1, 60, n).astype(np.int32)
    o = rng.integers(1, 300, n).astype(np.int32)
    if equal:
        s[:], o[:] = rng.choice([10, 20], n), rng.choice([40, 41], n)
    M = int((s + o).max()) + 700
    policies = [(planner, period, window, ratio) for planner, window in ((3, 300), (3, 40), (1, 0), (0, 0)) for ratio in RATIOS]
    print(f"online, quiet arrivals: {rate} a round, period {period}, equal {equal}, M={M}", flush=True)
    comp, stats, status = _run(a, s, o, M, policies)
    assert status == 0
    for k, c in enumerate(policies):
        _, c_o, st_o = oracle.online(a, s, o, M, *c)
        assert tuple(int(x) for x in stats[k]) == st_o, c
        assert (comp[k * n : (k + 1) * n] == c_o).all(), c


@pytest.mark.parametrize("where", [70, 99, 130])
def test_a_faulty_request_among_them_is_reported(where):
    from paper_2508_06133_amd import kvsched

    n, M = 150, 500
    a = np.arange(n, dtype=np.int32)
    s, o = np.full(n, 10, dtype=np.int32), np.full(n, 400, dtype=np.int32)
    s[where] = 0
    print(f"online, quiet arrivals: request {where} is faulty", flush=True)
    _, stats, status = _run(a, s, o, M, [(3, 100000, 300, (1, 1)), (1, 100000, 0, (1, 0))])
    assert (stats == -1).all() and status == kvsched.DEV_BAD_LENGTH
