"""GPU parity with the CPU oracle of orders placed a lane each where the start is found in one pass over the completions: budgets from one
request to all of them, lengths with many equal completion rounds, requests of one round among long ones, and the numbers of orders around
the line from which orders of more than eight requests take that way."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _lengths(rng, kind, n):
    if kind == "equal":
        return rng.integers(1, 3, n), rng.integers(1, 4, n)
    if kind == "steps":
        return rng.integers(1, 40, n), 8 * rng.integers(1, 6, n)
    if kind == "long":
        return rng.choice([1, 2000], n), rng.choice([1, 2, 900], n)
    return rng.integers(1, 200, n), rng.integers(1, 300, n)


@pytest.mark.parametrize("kind", ["equal", "steps", "long", "any"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 16, 17, 21, 31, 32])
def test_budgets(n, kind):
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    rows = 130 if n <= 8 else 512 * n
    orders = np.argsort(rng.random((rows, n)), axis=1).astype(np.int32)
    d_orders = torch.from_numpy(orders).to("cuda:0")
    some = np.r_[0:32, rows - 34:rows]
    ctx = kvsched.Context(0)
    try:
        for turn in range(3):
            s, o = (x.astype(np.int32) for x in _lengths(rng, kind, n))
            least, total = int((s + o).max()), int((s + o).sum())
            for M in sorted({least, least + 1, least + total // 8, least + total // 4, max(least, total // 2), max(least, total - 1)}):
                print(f"short rows, one pass: {kind} n={n} rows={rows} M={M}", flush=True)
                args = torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0"), M
                tel, comp = ctx.simulate(d_orders, *args)
                assert ctx.device_status() == 0
                tel_o, comp_o = oracle.simulate_many(s, o, M, orders[some])
                assert (tel.cpu().numpy()[some] == tel_o).all() and (comp.cpu().numpy()[some] == comp_o).all()
                if n > 8:  # one order fewer: a wavefront each
                    tel_w, comp_w = ctx.simulate(d_orders[1:], *args)
                    assert torch.equal(tel_w, tel[1:]) and torch.equal(comp_w, comp[1:])
    finally:
        ctx.close()
