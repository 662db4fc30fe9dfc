"""GPU parity with the CPU oracle of orders placed a lane per completion round (few decode lengths, up to long ones): numbers of
positions around the four a lane takes, its groups and chunks, budgets of one request and of many, tokens that are summed in
larger units, rows with more completions ahead than lanes, rows that are no permutations and lengths that cannot be scheduled."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda:0")


def _orders(rng, s, o, M, rows):
    """The base order, neighbours of it by a few exchanges, and random permutations."""
    n = len(s)
    base = oracle.sortedF(s, o, M)[0]
    orders = np.stack([base if r % 3 else rng.permutation(n) for r in range(rows)]).astype(np.int32)
    orders[0] = base
    for r in range(rows):
        for _ in range(r % 5):
            i, j = rng.integers(0, n, 2)
            orders[r, i], orders[r, j] = orders[r, j], orders[r, i]
    return orders


def _lengths(rng, what, n):
    if what == "bimodal":
        s = np.where(rng.random(n) < 0.5, 1, 4096)
        o = np.where(rng.random(n) < 0.5, 4096, 1)
        return s, o, 12288 + 40 * n
    if what == "tight":  # a budget of one request and a half
        s = rng.integers(1, 4000, n)
        return s, rng.choice([1, 7, 4096], n), 12288
    if what == "units":  # sums of a group's sizes do not fit 32 bits
        s = rng.integers(1, 1 << 25, n)
        return s, rng.choice([3, 2500], n), (1 << 29) + 77
    # four lengths whose sums hardly ever coincide, room for hundreds: some rows have more than 64 completions ahead
    s = rng.integers(1, 3000, n)
    return s, rng.choice([2100, 2213, 3001, 4096], n), 6000 + 400 * min(n, 2000)


@pytest.mark.parametrize("what", ["bimodal", "tight", "units", "many"])
@pytest.mark.parametrize("n,rows", [(1, 3), (4, 9), (63, 70), (64, 5), (65, 6), (255, 6), (257, 7), (512, 6), (513, 5), (1025, 6), (2500, 5),
                                    (8192, 2), (15873, 2)])
def test_orders(n, rows, what):
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n + rows)
    s, o, M = _lengths(rng, what, n)
    if n > 3:
        o[:4] = o.max()  # (long enough for the kernel to be chosen)
    s, o = s.astype(np.int32), o.astype(np.int32)
    orders = _orders(rng, s, o, M, rows)
    tel_o, comp_o = oracle.simulate_many(s, o, M, orders)
    for bound in (0, 4096):
        ctx = kvsched.Context(0)
        try:
            ctx.set_o_max(bound)
            for call in range(3):  # (the first may not know that the lengths are few)
                print(f"event rows: n={n} rows={rows} {what} bound={bound} call={call}", flush=True)
                tel, comp = ctx.simulate(_dev(orders), _dev(s), _dev(o), M)
                only, _ = ctx.simulate(_dev(orders), _dev(s), _dev(o), M, completions=False)
                assert ctx.device_status() == 0
                assert (tel.cpu().numpy() == tel_o).all() and (comp.cpu().numpy() == comp_o).all() and (only == tel).all()
        finally:
            ctx.close()


@pytest.mark.parametrize("n", [20, 100, 300, 1500, 2500])
def test_faulty(n):
    """A row that is no permutation and lengths that cannot be scheduled void their rows alone, and are reported."""
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    s, o, M = _lengths(rng, "bimodal", n)
    o[:2] = 1, 4096
    s, o = s.astype(np.int32), o.astype(np.int32)
    orders = _orders(rng, s, o, M, 9)
    good = [0, 1, 4, 7, 8]
    orders[2, n - 1] = orders[2, 0]
    orders[3, n // 2] = -1
    orders[5, 1] = n
    orders[6, 0] = 2**31 - 1
    tel_o, comp_o = oracle.simulate_many(s, o, M, orders[good])
    for bound in (0, 4096):
        ctx = kvsched.Context(0)
        try:
            ctx.set_o_max(bound)
            for what in ("row", "row", "s", "row", "o", "long", "good", "row"):
                print(f"event rows, faulty: n={n} bound={bound} {what}", flush=True)
                s1, o1, rows = s.copy(), o.copy(), orders if what == "row" else orders[good]
                if what == "s":
                    s1[n - 1] = 0
                if what == "o":
                    o1[n // 2] = 0
                if what == "long":
                    o1[n // 2] = 5000
                tel, comp = ctx.simulate(_dev(rows), _dev(s1), _dev(o1), M)
                status = ctx.device_status()
                tel, comp = tel.cpu().numpy(), comp.cpu().numpy()
                if what == "row":
                    assert status == kvsched.DEV_BAD_ORDER and (np.delete(tel, good) == -1).all()
                    assert (tel[good] == tel_o).all() and (comp[good] == comp_o).all()
                elif what == "good":
                    assert status == 0 and (tel == tel_o).all() and (comp == comp_o).all()
                elif what == "long":
                    if bound:
                        assert status == kvsched.DEV_O_MAX and (tel == -1).all()
                    else:
                        t1, c1 = oracle.simulate_many(s1, o1, M, orders[good])
                        assert status == 0 and (tel == t1).all() and (comp == c1).all()
                else:
                    assert status == kvsched.DEV_BAD_LENGTH and (tel == -1).all()
        finally:
            ctx.close()


@pytest.mark.parametrize("lengths", ["few", "many"])
@pytest.mark.parametrize("n", [33, 100, 127, 577, 1500, 8193, 8255])
def test_faulty_last_position(n, lengths):
    """A row whose LAST id is none: the lanes past the end of the row, which take that position's id, read nothing by it.  Many lengths: the
    kernel is launched and leaves the rows to the timeline kernel (from 8192 positions on by itself, else because the call before had few)."""
    from paper_2508_06133_amd import kvsched

    assert n % 64 != 0
    rng = np.random.default_rng(n)
    s, o, M = _lengths(rng, "bimodal", n)
    o[:2] = 1, 4096
    few = o.astype(np.int32)
    if lengths == "many":
        o = rng.integers(1, 400, n)
        o[:2] = 1, 4096
    s, o = s.astype(np.int32), o.astype(np.int32)
    orders = _orders(rng, s, o, M, 5)
    orders[1, n - 1] = -1
    orders[2, n - 1] = n
    orders[3, n - 1] = 2**31 - 1
    good = [0, 4]
    tel_o, comp_o = oracle.simulate_many(s, o, M, orders[good])
    for bound in (0, 4096):
        ctx = kvsched.Context(0)
        try:
            ctx.set_o_max(bound)
            for call in range(2):
                print(f"event rows, last id: n={n} {lengths} bound={bound} call={call}", flush=True)
                ctx.simulate(_dev(orders[good]), _dev(s), _dev(few), M)
                tel, comp = ctx.simulate(_dev(orders), _dev(s), _dev(o), M)
                assert ctx.device_status() == kvsched.DEV_BAD_ORDER
                tel, comp = tel.cpu().numpy(), comp.cpu().numpy()
                assert (tel[[1, 2, 3]] == -1).all() and (tel[good] == tel_o).all() and (comp[good] == comp_o).all()
                only, _ = ctx.simulate(_dev(orders), _dev(s), _dev(o), M, completions=False)
                assert (only.cpu().numpy() == tel).all()
        finally:
            ctx.close()


@pytest.mark.parametrize("bound", [0, 4096])
def test_rows_that_would_be_resumed(bound):
    """Rows that would be resumed are placed a lane per completion round where this call's lengths are known to be few, whatever those of the call
    before were: without a bound from the caller (several workgroups look them over); with one they are always resumed."""
    from paper_2508_06133_amd import kvsched

    n, rows = 4500, 4096
    rng = np.random.default_rng(7)
    s, few, M = _lengths(rng, "bimodal", n)
    many = rng.integers(1, 400, n)
    few[:2] = many[:2] = 1, 4096
    base = rng.permutation(n).astype(np.int32)
    orders = np.tile(base, (rows, 1))
    for r in range(1, rows):
        i, j = rng.integers(64, n, 2)
        orders[r, i], orders[r, j] = orders[r, j], orders[r, i]
    d_orders, d_s, lengths = _dev(orders), _dev(s), {"few": _dev(few), "many": _dev(many)}
    ctx, plain = kvsched.Context(0), kvsched.Context(0)
    try:
        plain.set_resume_min_rows(0)
        ctx.set_o_max(bound)
        want = {k: plain.simulate(d_orders, d_s, o, M) for k, o in lengths.items()}
        for call, which in enumerate(["few", "many", "few", "few", "many", "many", "few", "few", "few", "many"]):
            print(f"event rows, would be resumed: bound={bound} call {call} {which}", flush=True)
            tel, comp = ctx.simulate(d_orders, d_s, lengths[which], M)
            assert bool((tel == want[which][0]).all()) and bool((comp == want[which][1]).all()) and ctx.device_status() == 0
            resumed = bool((ctx.simulate_resume_positions(rows) > 0).any())
            assert resumed == (bound > 0 or which == "many")
        for k, o in (("few", few), ("many", many)):  # the plain context itself, a few rows against the oracle
            t, c = oracle.simulate_many(s.astype(np.int32), o.astype(np.int32), M, orders[:3])
            assert (want[k][0][:3].cpu().numpy() == t).all() and (want[k][1][:3].cpu().numpy() == c).all()
    finally:
        ctx.close()
        plain.close()


@pytest.mark.parametrize("n,rows,differs,budget,resumed", [(2100, 4096, 0.9, 12288, True), (2100, 4096, 0.1, 12288, False), (2100, 4096, 0.9, 1 << 19, False),
                                                           (2100, 4096, 0.65, 12288, False), (2100, 4096, 0.67, 12288, True), (403, 20500, 0.9, 12288, True)])
def test_rows_that_differ_late(n, rows, differs, budget, resumed):
    """Without a bound, rows that agree with row 0 over two thirds and more are resumed where the budget is small, though their lengths are
    few; the number of the length scan and of the look at the rows that follows it are told apart over several calls."""
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    o = rng.choice([500, 1000, 2000, 2500], n)
    o[0] = 2500
    s = rng.integers(1, 3000, n)
    orders = np.tile(rng.permutation(n).astype(np.int32), (rows, 1))
    lo = int(differs * n)
    for r in range(1, rows):
        j = rng.integers(lo + 1, n)
        orders[r, lo], orders[r, j] = orders[r, j], orders[r, lo]
    d_orders, d_s, d_o = _dev(orders), _dev(s), _dev(o)
    ctx, plain = kvsched.Context(0), kvsched.Context(0)
    try:
        plain.set_resume_min_rows(0)
        want = plain.simulate(d_orders, d_s, d_o, budget)
        for call in range(3):
            print(f"event rows, differ late: n={n} rows={rows} from {differs} budget={budget} call {call}", flush=True)
            tel, comp = ctx.simulate(d_orders, d_s, d_o, budget)
            assert bool((tel == want[0]).all()) and bool((comp == want[1]).all()) and ctx.device_status() == 0
            assert bool((ctx.simulate_resume_positions(rows) > 0).any()) == resumed
        t, c = oracle.simulate_many(s.astype(np.int32), o.astype(np.int32), budget, orders[:3])
        assert (tel[:3].cpu().numpy() == t).all() and (comp[:3].cpu().numpy() == c).all()
    finally:
        ctx.close()
        plain.close()
