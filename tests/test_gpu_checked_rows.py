"""GPU parity with the CPU oracle of orders of up to 1024 requests, which the timeline kernel checks and writes by request id
itself: sizes around a block and the limit, one and many rows, every register file, with and without a bound from the
caller, and orders that are no permutations beside lengths that cannot be scheduled."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows,longest", [(n, rows, longest) for longest in (100, 500, 2000, 4000, 8000, 14000, 15000)
                                            for n, rows in ((9, 1), (31, 5), (63, 1), (64, 1), (64, 300), (65, 3))]
                         + [(130, 3, 2000), (256, 40, 100), (1023, 2, 100), (1024, 70, 500), (1024, 3, 1500), (1025, 2, 500)])
def test_rows(n, rows, longest):
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n + longest)
    s, o = rng.integers(1, 500, n).astype(np.int32), rng.integers(1, longest // 4 + 2, n).astype(np.int32)
    o[n // 3] = longest
    M = int((s + o).max()) + 2000
    orders = np.argsort(rng.random((rows, n)), axis=1).astype(np.int32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    ctx = kvsched.Context(0)
    try:
        print(f"one block: n={n} rows={rows} decodes up to {longest}", flush=True)
        check = list(range(min(rows, 8))) + [rows - 1]
        tel_o, comp_o = oracle.simulate_many(s, o, M, orders[check])
        for bound in (0, 0, longest, 16384):  # (the second call without a bound takes the first one's file for granted)
            ctx.set_o_max(bound)
            tel, comp = ctx.simulate(dev(orders), dev(s), dev(o), M)
            assert ctx.device_status() == 0
            assert (tel.cpu().numpy()[check] == tel_o).all() and (comp.cpu().numpy()[check] == comp_o).all()
        ctx.set_o_max(0)
        for at, value in ((0, -1), (n - 1, n), (n // 2, 2**31 - 1), (1, int(orders[rows // 2, 0])), (n - 2, -2**31)):
            bad = orders.copy()
            bad[rows // 2, at] = value
            tel, comp = ctx.simulate(dev(bad), dev(s), dev(o), M)
            assert ctx.device_status() == kvsched.DEV_BAD_ORDER
            tel = tel.cpu().numpy()
            assert tel[rows // 2] == -1
            if rows > 2:
                assert tel[rows - 1] == tel_o[-1] and (comp[rows - 1].cpu().numpy() == comp_o[-1]).all()
        wrong = s.copy()
        wrong[n // 2] = M
        tel, _ = ctx.simulate(dev(bad), dev(wrong), dev(o), M, completions=False)
        assert ctx.device_status() == kvsched.DEV_BAD_ORDER | kvsched.DEV_BAD_LENGTH and (tel == -1).all()
    finally:
        ctx.close()
