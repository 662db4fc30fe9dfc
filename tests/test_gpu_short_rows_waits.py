"""GPU parity with the CPU oracle of orders placed a lane each in which requests of a few rounds wait for long ones: budgets
that one or two of the long ones fill, exactly or with a few tokens left."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows", [(3, 65), (8, 128), (16, 8200), (32, 32769)])
@pytest.mark.parametrize("s_long,o_long,room", [(4096, 4096, 0), (4096, 4096, 1), (100, 700, 801), (1, 4096, 4096), (300, 900, 40)])
def test_short_behind_long(n, rows, s_long, o_long, room):
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n + s_long + room)
    s = np.where(rng.random(n) < 0.5, 1, s_long).astype(np.int32)
    o = np.where(rng.random(n) < 0.5, rng.integers(1, 4, n), o_long).astype(np.int32)
    s[0], o[0] = s_long, o_long
    M = s_long + o_long + room
    orders = np.argsort(rng.random((rows, n)), axis=1).astype(np.int32)
    print(f"short rows, waits: n={n} rows={rows} s={s_long} o={o_long} M={M}", flush=True)
    ctx = kvsched.Context(0)
    try:
        d = [torch.from_numpy(x).to("cuda:0") for x in (orders, s, o)]
        tel, comp = ctx.simulate(d[0], d[1], d[2], M)
        assert ctx.device_status() == 0
    finally:
        ctx.close()
    check = np.unique(np.concatenate([np.arange(6), rng.integers(0, rows, 6), [rows - 1]]))
    tel_o, comp_o = oracle.simulate_many(s, o, M, orders[check])
    assert (tel.cpu().numpy()[check] == tel_o).all() and (comp.cpu().numpy()[check] == comp_o).all()
