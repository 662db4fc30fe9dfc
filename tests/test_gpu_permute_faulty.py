"""Rows that are no permutations where the completion rounds are put in order by request id in a pass of their own (a declared
prefix, orders of more than 1024 requests): the requests that a row leaves out complete in round -1, other rows are unharmed."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows,prefix", [(70, 41, 64), (129, 15, 65), (256, 5, 64), (257, 9, 128), (1025, 6, 0), (3000, 5, 0)])
def test_requests_that_do_not_occur(n, rows, prefix):
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    s, o = rng.integers(1, 200, n).astype(np.int32), rng.integers(1, 300, n).astype(np.int32)
    orders = np.argsort(rng.random((rows, n)), axis=1).astype(np.int32)
    orders[:, :prefix] = np.arange(prefix)
    for row in orders:  # (still permutations, of one prefix)
        rest = np.setdiff1d(np.arange(n), np.arange(prefix))
        row[prefix:] = rng.permutation(rest)
    faulty = [1, rows - 1]
    left_out = [int(orders[r, n - 1]) for r in faulty]
    for r in faulty:
        orders[r, n - 1] = orders[r, n - 2]
    print(f"rows by request id, faulty: n={n} rows={rows} prefix={prefix}", flush=True)
    ctx = kvsched.Context(0)
    try:
        d = [torch.from_numpy(x).to("cuda:0") for x in (orders, s, o)]
        tel, comp = ctx.simulate(d[0], d[1], d[2], 4000, common_prefix=prefix)
        assert ctx.device_status() == 2
    finally:
        ctx.close()
    tel, comp = tel.cpu().numpy(), comp.cpu().numpy()
    assert (tel[faulty] == -1).all()
    for r, request in zip(faulty, left_out):
        assert comp[r, request] == -1 and (comp[r] == -1).sum() == 1
    whole = np.setdiff1d(np.arange(rows), faulty)[:3]
    tel_o, comp_o = oracle.simulate_many(s, o, 4000, orders[whole])
    assert (tel[whole] == tel_o).all() and (comp[whole] == comp_o).all()
