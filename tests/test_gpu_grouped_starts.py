"""Requests that start in one round many at a time: bursts longer than a block of 64 positions and longer than the kernel's
list, windows that end at the edges of rows and of chunks of four rows, budgets so large that sizes are counted in
coarser units, bursts behind round 0, saved states taken and resumed inside a burst."""
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


def check(ctx, s, o, M, orders, rows=None):
    import torch

    tel, comp = ctx.simulate(torch.from_numpy(orders).cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(o).cuda(), M)
    tel, comp = tel.cpu().numpy(), comp.cpu().numpy()
    for row in range(len(orders)) if rows is None else rows:
        _, want, total = oracle.simulate(s, o, M, orders[row], literal=False)[:3]
        assert tel[row] == total and (comp[row] == np.asarray(want)).all(), row
    assert ctx.device_status() == 0


def lengths(rng, kind, n, o_max):
    if kind == "edges":
        ends = [64 * r + d for r in (1, 3, 4, 5, 8, 16, 31, 32, 60, 64, 124, 128, 220, 224) for d in (-1, 0, 1)]
        o = rng.choice([e for e in ends if 1 <= e <= o_max], n)
    elif kind == "bimodal":
        o = np.where(rng.random(n) < 0.5, 1, o_max)
    else:
        o = rng.integers(1, o_max + 1, n)
    o = o.astype(np.int32)
    o[rng.integers(0, n)] = o_max
    return o


@pytest.mark.parametrize("o_max", [512, 2048, 4096, 8192, 14336])
@pytest.mark.parametrize("kind", ["edges", "bimodal", "uniform"])
@pytest.mark.parametrize("n", [16, 129, 700])
def test_bursts(ctx, o_max, kind, n):
    """Budgets for a quarter of the requests, for all but a few, for all of them."""
    print(f"o_max={o_max} {kind} n={n}", flush=True)
    rng = np.random.default_rng(o_max + n)
    o = lengths(rng, kind, n, o_max)
    s = rng.integers(1, 900, n).astype(np.int32)
    orders = np.stack([np.argsort(s + o, kind="stable")] + [rng.permutation(n)]).astype(np.int32)
    ctx.set_o_max(o_max)
    total = int((s.astype(np.int64) + o).sum())
    largest = int((s + o).max())
    for M in (largest, max(largest, total // 4), max(largest, total - 5 * largest), total, total + 7):
        check(ctx, s, o, M, orders)


@pytest.mark.parametrize("M_bits", [25, 26, 28, 29])
def test_sizes_in_coarser_units(ctx, M_bits):
    print(f"M_bits={M_bits}", flush=True)
    rng = np.random.default_rng(M_bits)
    n = 400
    o = rng.integers(1, 700, n).astype(np.int32)
    M = (1 << M_bits) + int(rng.integers(0, 1000))
    s = (rng.integers(1, M // 12, n)).astype(np.int32)
    s[::7] = rng.integers(1, 50, len(s[::7]))
    s[3] = M - int(o[3])
    orders = np.stack([np.argsort(s + o, kind="stable")] + [rng.permutation(n) for _ in range(3)]).astype(np.int32)
    ctx.set_o_max(0)
    check(ctx, s, o, M, orders)


@pytest.mark.parametrize("o_max", [2048, 4096, 8192])
@pytest.mark.parametrize("completions", [True, False])
def test_states_saved_and_resumed_inside_a_burst(ctx, o_max, completions):
    import torch

    print(f"o_max={o_max} completions={completions}", flush=True)
    rng = np.random.default_rng(o_max)
    n, rows = 900, 96
    o = lengths(rng, "uniform", n, o_max)
    o[rng.random(n) < 0.6] //= 16
    o = np.maximum(o, 1)
    s = rng.integers(1, 900, n).astype(np.int32)
    M = int((s.astype(np.int64) + o).sum() * 0.4)
    base = np.argsort(s + o, kind="stable").astype(np.int32)
    orders = np.repeat(base[None], rows, 0)
    for r in range(1, rows):
        i, j = rng.integers(0, n, 2)
        orders[r, i], orders[r, j] = orders[r, j], orders[r, i]
    moves = np.concatenate([[[0, 0, 0]], np.stack([rng.integers(0, 2, rows), rng.integers(0, n, rows), rng.integers(0, n, rows)], 1)])
    moves = moves.astype(np.int32)
    tel_o, comp_o = oracle.simulate_many(s, o, M, orders, literal=False)
    tel_mo, res_o = oracle.best_neighbor(s, o, M, base, moves, literal=False)
    d = [torch.from_numpy(x).cuda() for x in (orders, s, o, base, moves)]
    ctx.set_o_max(o_max)
    ctx.set_resume_min_rows(2)
    try:
        for polls in (4096, 0):
            ctx.set_resume_one_launch(polls)
            tel, comp = ctx.simulate(d[0], d[1], d[2], M, completions)
            assert (tel.cpu().numpy() == tel_o).all()
            assert not completions or (comp.cpu().numpy() == comp_o).all()
            tel_m, res = ctx.best_neighbor(d[3], d[4], d[1], d[2], M)
            assert (tel_m.cpu().numpy() == tel_mo).all() and tuple(int(x) for x in res.cpu().numpy()) == res_o
        prefix = np.repeat(base[None], 8, 0)  # a declared prefix that ends inside the burst, off the blocks of 64
        for r in range(1, 8):
            prefix[r, 200:] = base[200:][rng.permutation(n - 200)]
        tel, comp = ctx.simulate(torch.from_numpy(prefix).cuda(), d[1], d[2], M, completions, common_prefix=200)
        tel_p, comp_p = oracle.simulate_many(s, o, M, prefix, literal=False)
        assert (tel.cpu().numpy() == tel_p).all()
        assert not completions or (comp.cpu().numpy() == comp_p).all()
    finally:
        ctx.set_resume_one_launch(4096)
        ctx.set_resume_min_rows(-1)
    assert ctx.device_status() == 0


def test_a_long_backlog_in_few_bursts(ctx):
    """Bursts of several hundred requests behind round 0 (the kernel's list fills up), completion rounds scattered by id."""
    print("long backlog", flush=True)
    rng = np.random.default_rng(8)
    n = 20000
    s = np.where(rng.random(n) < 0.5, 1, 4096).astype(np.int32)
    o = np.where(rng.random(n) < 0.5, 4096, 1).astype(np.int32)
    M = 420000 * 4
    base = np.lexsort((np.arange(n), o, s + o)).astype(np.int32)
    orders = np.stack([base, base.copy(), rng.permutation(n)]).astype(np.int32)
    for _ in range(64):
        i, j = rng.integers(0, n, 2)
        orders[1, i], orders[1, j] = orders[1, j], orders[1, i]
    ctx.set_o_max(4096)
    check(ctx, s, o, M, orders)
