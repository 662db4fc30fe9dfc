"""Orders placed a lane each that cannot be scheduled: a budget of one token, which no request fits, requests that hold more
than any budget beside others that wait for one another, and rows that are no permutations.  The CPU oracle refuses them; the
rows report -1."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 130), (2, 64), (8, 65), (9, 8192), (16, 8200), (17, 32768), (32, 32770)]  # (requests, orders)


def _run(s, o, M, orders, bound=0):
    import torch
    from paper_2508_06133_amd import kvsched

    ctx = kvsched.Context(0)
    try:
        ctx.set_o_max(bound)
        d = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to("cuda:0") for x in (orders, s, o)]
        tel, comp = ctx.simulate(d[0], d[1], d[2], M)
        status = ctx.device_status()
        return tel.cpu().numpy(), comp.cpu().numpy(), status
    finally:
        ctx.close()


def _orders(rng, n, rows):
    return np.argsort(rng.random((rows, n)), axis=1).astype(np.int32)


@pytest.mark.parametrize("bound", [0, 4])
@pytest.mark.parametrize("n,rows", SIZES)
def test_budget_of_one_token(n, rows, bound):
    rng = np.random.default_rng(n)
    s, o = rng.integers(1, 5, n), rng.integers(1, 5, n)
    print(f"short rows, M=1: n={n} rows={rows} bound={bound}", flush=True)
    tel, _, status = _run(s, o, 1, _orders(rng, n, rows), bound)
    assert status == 1 and (tel == -1).all()


@pytest.mark.parametrize("n,rows", SIZES)
def test_budget_of_two_tokens(n, rows):
    """The least budget that holds a request: one runs after the other."""
    rng = np.random.default_rng(n)
    orders = _orders(rng, n, rows)
    print(f"short rows, M=2: n={n} rows={rows}", flush=True)
    tel, comp, status = _run(np.ones(n), np.ones(n), 2, orders)
    assert status == 0 and (tel == n * (n + 1) // 2).all()
    assert (np.take_along_axis(comp, orders.astype(np.int64), axis=1) == np.arange(1, n + 1)).all()


@pytest.mark.parametrize("n,rows", SIZES[2:])
def test_unschedulable_among_others(n, rows):
    rng = np.random.default_rng(n)
    s, o = rng.integers(1, 3000, n), rng.integers(1, 2048, n)
    M = int((s + o).max()) + 100
    orders = _orders(rng, n, rows)
    for value in (0, -2**31, M, 2**31 - 1):
        bad = s.copy()
        bad[rng.integers(0, n)] = value
        print(f"short rows, unschedulable: n={n} rows={rows} s={value}", flush=True)
        tel, _, status = _run(bad, o, M, orders)
        assert status == 1 and (tel == -1).all()
    few = orders[:4]
    tel, comp, status = _run(s, o, M, orders)
    tel_o, comp_o = oracle.simulate_many(s.astype(np.int32), o.astype(np.int32), M, few)
    assert status == 0 and (tel[:4] == tel_o).all() and (comp[:4] == comp_o).all()


@pytest.mark.parametrize("n,rows", SIZES[2:])
def test_requests_that_do_not_occur(n, rows):
    """A row that names one request twice, or one that does not exist: the completion round of those it leaves out is -1."""
    rng = np.random.default_rng(n)
    s, o = rng.integers(1, 9, n), rng.integers(1, 9, n)
    orders = _orders(rng, n, rows)
    left_out = {0: orders[0, 0], rows // 2: orders[rows // 2, n - 1], rows - 1: orders[rows - 1, 1]}
    orders[0, 0], orders[rows // 2, n - 1], orders[rows - 1, 1] = orders[0, 1], orders[rows // 2, 0], 2**31 - 1
    left_out[rows - 1] = None if left_out[rows - 1] == n - 1 else left_out[rows - 1]  # (read as request n - 1)
    print(f"short rows, requests left out: n={n} rows={rows}", flush=True)
    tel, comp, status = _run(s, o, 40, orders)
    assert status == 2 and (tel[list(left_out)] == -1).all() and (tel == -1).sum() == 3
    for row, request in left_out.items():
        assert (comp[row] == -1).sum() == (request is not None) and (request is None or comp[row, request] == -1)
    whole = np.setdiff1d(np.arange(rows), list(left_out))[:4]
    tel_o, comp_o = oracle.simulate_many(s.astype(np.int32), o.astype(np.int32), 40, orders[whole])
    assert (tel[whole] == tel_o).all() and (comp[whole] == comp_o).all()


def _placed(s, o, M, order):
    """Completion rounds by request, round by round; a request that cannot be scheduled ends where it is reached."""
    memory, t, done = np.zeros(1 + int(np.maximum(o, 0).sum()), dtype=np.int64), 0, np.zeros(len(order), dtype=np.int64)
    for i in order:
        good = s[i] >= 1 and o[i] >= 1 and s[i] + o[i] <= M
        held = int(s[i]) + 1 + np.arange(o[i]) if good else np.zeros(0, dtype=np.int64)
        while (memory[t + 1 : t + 1 + len(held)] + held > M).any():
            t += 1
        memory[t + 1 : t + 1 + len(held)] += held
        done[i] = t + len(held)
    return done


@pytest.mark.parametrize("n,rows", [(3, 70), (8, 130), (16, 8192), (32, 16384)])
def test_unschedulable_takes_no_rounds(n, rows):
    """Budgets that a request or two fill, so that others start where one completes: those behind an unschedulable request are placed
    as if it were not there."""
    rng = np.random.default_rng(n)
    orders = _orders(rng, n, rows)
    some = np.r_[0:12, rows - 12:rows]
    for turn in range(6):
        s, o = rng.integers(1, 10, n), rng.integers(1, 7, n)
        M = 14 if turn % 2 else 16
        if n == 3:
            s, o, M = np.array([5, 8, 1]), np.array([5, 4, 1]), 14
            orders[0] = 0, 1, 2
        bad = n - 1 if n == 3 else rng.integers(0, n)
        s[bad] = M + turn
        print(f"short rows, placed around an unschedulable one: n={n} rows={rows} M={M} turn={turn}", flush=True)
        tel, comp, status = _run(s, o, M, orders)
        assert status == 1 and (tel == -1).all()
        for row in some:
            assert (comp[row] == _placed(s, o, M, orders[row])).all(), (turn, row)
