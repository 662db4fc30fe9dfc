"""GPU parity with the CPU oracle of orders placed a lane each: numbers of requests around 8, 16 and 32, numbers of orders
around a wavefront's 64 and the lines from which longer orders take that way, the longest decodes, a budget that
one request fills, orders that are no permutations and lengths that cannot be scheduled."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _run(s, o, M, orders, bound=0):
    import torch
    from paper_2508_06133_amd import kvsched

    ctx = kvsched.Context(0)
    try:
        ctx.set_o_max(bound)
        d = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to("cuda:0") for x in (orders, s, o)]
        tel, comp = ctx.simulate(d[0], d[1], d[2], M)
        only, none = ctx.simulate(d[0], d[1], d[2], M, completions=False)
        status = ctx.device_status()
        assert none is None and (only == tel).all()
        return tel.cpu().numpy(), comp.cpu().numpy(), status
    finally:
        ctx.close()


@pytest.mark.parametrize("lengths", ["tiny", "mixed", "longest"])
@pytest.mark.parametrize("n,rows", [(1, 1), (1, 65), (2, 64), (7, 63), (8, 1), (8, 129), (9, 8191), (9, 8192), (15, 8193), (16, 8192),
                                    (17, 32768), (24, 32767), (32, 32769), (33, 32768)])
def test_orders(n, rows, lengths):
    rng = np.random.default_rng(100 * n + rows)
    if lengths == "tiny":
        s, o = rng.integers(1, 9, n), rng.integers(1, 9, n)
        M = int((s + o).max()) + n
    elif lengths == "mixed":
        s, o = rng.integers(1, 3000, n), rng.integers(1, 2048, n)
        M = int((s + o).max()) + 1500
    else:
        s, o = rng.integers(1, 20000, n), rng.integers(15000, 16385, n)
        M = int((s + o).max())
    s, o = s.astype(np.int32), o.astype(np.int32)
    orders = np.argsort(rng.random((rows, n)), axis=1).astype(np.int32)
    print(f"short rows: n={n} rows={rows} {lengths} M={M}", flush=True)
    tel, comp, status = _run(s, o, M, orders, bound=16384 if rows % 2 else 0)
    check = np.unique(np.concatenate([np.arange(min(rows, 130)), rng.integers(0, rows, 200), [rows - 1]]))
    if lengths == "longest":  # (up to a second an order in the oracle, which goes from round to round)
        check = np.unique([0, rows - 1])
    tel_o, comp_o = oracle.simulate_many(s, o, M, orders[check])
    assert status == 0 and (tel[check] == tel_o).all() and (comp[check] == comp_o).all()


@pytest.mark.parametrize("n", [3, 8, 16])
def test_malformed(n):
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    rows = 8200
    s, o, M = rng.integers(1, 9, n).astype(np.int32), rng.integers(1, 9, n).astype(np.int32), 40
    orders = np.argsort(rng.random((rows, n)), axis=1).astype(np.int32)
    void = [0, 63, 64, rows - 1]
    orders[0, 0], orders[63, n - 1], orders[rows - 1, 1] = -1, n, 2**31 - 1
    orders[64, 0] = orders[64, 1]
    good = np.setdiff1d(np.arange(rows), void)
    print(f"short rows, malformed: n={n}", flush=True)
    tel, comp, status = _run(s, o, M, orders)
    tel_o, comp_o = oracle.simulate_many(s, o, M, orders[good])
    assert status == kvsched.DEV_BAD_ORDER and (tel[void] == -1).all()
    assert (tel[good] == tel_o).all() and (comp[good] == comp_o).all()
    for which, value, bound, bit in (("s", 0, 0, 1), ("o", 0, 0, 1), ("s", M, 0, 1), ("o", 9, 8, 8)):
        bad_s, bad_o = s.copy(), o.copy()
        (bad_s if which == "s" else bad_o)[n // 2] = value
        tel, _, status = _run(bad_s, bad_o, M, orders[good], bound)
        assert status == bit and (tel == -1).all()
