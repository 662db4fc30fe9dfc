"""GPU parity of the passes around the timelines at the sizes where they split their work differently: rows permuted
several to a workgroup, the argmin and the length scan over one or many workgroups."""
import numpy as np
import pytest

import oracle
from paper_2508_06133_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2508_06133_amd import kvsched

    c = kvsched.Context(0)
    yield c
    c.close()


def _dev(a, dtype=np.int32):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).to("cuda:0")


@pytest.mark.parametrize("n", [1, 2, 31, 33, 200, 255, 256, 257])
def test_short_rows(ctx, n):
    rng = np.random.default_rng(n)
    s, o = rng.integers(1, 9, n).astype(np.int32), rng.integers(1, 9, n).astype(np.int32)
    M = 40
    for C in (1, 2, 1024 // n, 1024 // n + 1, 130):
        if C < 1:
            continue
        print(f"short rows: n={n} C={C}", flush=True)
        rows = np.stack([rng.permutation(n) for _ in range(C)]).astype(np.int32)
        bad = C // 2 if C > 2 and n > 1 else None
        if bad is not None:
            rows[bad, 0] = rows[bad, 1]
        tel, comp = ctx.simulate(_dev(rows), _dev(s), _dev(o), M)
        tel, comp = tel.cpu().numpy(), comp.cpu().numpy()
        keep = np.arange(C) != (-1 if bad is None else bad)
        tel_o, comp_o = oracle.simulate_many(s, o, M, rows[keep], literal=False)
        assert (tel[keep] == tel_o).all() and (comp[keep] == comp_o).all()
        assert bad is None or tel[bad] == -1
        assert ctx.device_status() == (0 if bad is None else 2)


@pytest.mark.parametrize("K", [1, 63, 4096, 4097, 8193, 131071, 200000])
def test_argmin_over_many_workgroups(ctx, K):
    import torch

    rng = np.random.default_rng(K)
    for _ in range(3):
        tel = rng.integers(0, 50, K)
        tel[rng.random(K) < 0.3] = -1
        valid = np.flatnonzero(tel >= 0)
        want = (int(valid[np.argmin(tel[valid])]), int(tel[valid].min())) if len(valid) else (-1, -1)
        got = ctx.argmin(torch.from_numpy(tel.astype(np.int64)).to("cuda:0")).cpu().numpy()
        assert tuple(int(x) for x in got) == want
    assert tuple(ctx.argmin(torch.full((K,), -1, dtype=torch.int64, device="cuda:0")).cpu().tolist()) == (-1, -1)


@pytest.mark.parametrize("n", [4096, 4097, 20000])
def test_length_scan_over_many_workgroups(ctx, n):
    rng = np.random.default_rng(n)
    s, o = rng.integers(1, 40, n).astype(np.int32), rng.integers(1, 40, n).astype(np.int32)
    for where in (0, n // 2, n - 1):
        o2 = o.copy()
        o2[where] = 1900  # the longest decode decides which timeline kernel runs
        M = 9000
        row = rng.permutation(n).astype(np.int32)[None]
        tel, comp = ctx.simulate(_dev(row), _dev(s), _dev(o2), M)
        tel_o, comp_o = oracle.simulate_many(s, o2, M, row, literal=False)
        assert (tel.cpu().numpy() == tel_o).all() and (comp.cpu().numpy() == comp_o).all() and ctx.device_status() == 0
        o2[where] = 0
        tel, _ = ctx.simulate(_dev(row), _dev(s), _dev(o2), M)
        assert int(tel.item()) == -1 and ctx.device_status() & 1
    # moves: the lowest and highest position they touch decide what is placed once
    s, o, M = s[:600], o[:600], 900
    base = rng.permutation(600).astype(np.int32)
    moves = workloads.window_moves(rng, n, 200, 420)
    tel, res = ctx.best_neighbor(_dev(base), _dev(moves), _dev(s), _dev(o), M)
    pick = rng.integers(0, n, 200)
    rows = workloads.orders_from_moves(base, moves[pick])
    tel_o, _ = oracle.simulate_many(s, o, M, rows, literal=False)
    tel = tel.cpu().numpy()
    assert (tel[pick] == tel_o).all() and int(res[0].item()) == int(np.argmin(tel)) and ctx.device_status() == 0
