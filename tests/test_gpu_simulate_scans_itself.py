"""Calls of kvsched_simulate that have no length scan ahead of their timelines (orders of up to 256 requests): the status they
leave is their own, whatever the calls before and after left, and a wrong guess of the longest decode changes nothing."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda:0")


def _rows(rng, n, C, faulty):
    rows = np.stack([rng.permutation(n) for _ in range(C)]).astype(np.int32)
    if faulty:
        rows[C // 2, 0] = rows[C // 2, n - 1] if n > 1 else 5
    return rows


@pytest.mark.parametrize("n,C", [(1, 3), (8, 70), (63, 5), (64, 1), (65, 9), (255, 6), (256, 6), (257, 6), (20, 8200)])
@pytest.mark.parametrize("bound", [0, 300])
def test_status_is_that_of_the_last_call(n, C, bound):
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n + C)
    s, o = rng.integers(1, 100, n).astype(np.int32), rng.integers(1, 301, n).astype(np.int32)
    M = 1500
    ctx = kvsched.Context(0)
    try:
        ctx.set_o_max(bound)
        print(f"simulate without a scan: n={n} C={C} bound={bound}", flush=True)
        check = min(C, 6)
        # a good call, faulty rows, faulty lengths, decodes above the bound, a call with a scan between them
        for what in ("good", "row", "good", "length", "good", "row", "long", "sorted", "row", "good", "good"):
            rows = _rows(rng, n, C, what == "row")
            s1, o1 = s.copy(), o.copy()
            if what == "length":
                s1[n // 2] = 0
            if what == "long":
                o1[n // 2] = 310
            if what == "sorted":
                ctx.sortedF(_dev(s1), _dev(o1), M)
                assert ctx.device_status() == 0
                continue
            tel, comp = ctx.simulate(_dev(rows), _dev(s1), _dev(o1), M)
            status = ctx.device_status()
            tel, comp = tel.cpu().numpy(), comp.cpu().numpy()
            want = {"good": 0, "row": kvsched.DEV_BAD_ORDER, "length": kvsched.DEV_BAD_LENGTH,
                    "long": kvsched.DEV_O_MAX if bound else 0}[what]
            assert status == want, what
            if what in ("length",) or (what == "long" and bound):
                assert (tel == -1).all()
                continue
            good = [c for c in range(C) if what != "row" or c != C // 2][:check]
            if good:
                tel_o, comp_o = oracle.simulate_many(s1, o1, M, rows[good], literal=False)
                assert (tel[good] == tel_o).all() and (comp[good] == comp_o).all(), what
            if what == "row":
                assert tel[C // 2] == -1
    finally:
        ctx.close()


def test_wrong_guesses():
    """Backlogs whose longest decodes need other register files, the ring, or are out of range, in turn."""
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(3)
    ctx = kvsched.Context(0)
    try:
        for longest in (40, 600, 40, 3000, 5000, 600, 15000, 40, 14336, 17000, 40, 17000, 15000):
            n, C = 40, 20
            s, o = rng.integers(1, 50, n).astype(np.int32), rng.integers(1, 30, n).astype(np.int32)
            o[7] = longest
            M = 18000
            rows = _rows(rng, n, C, longest == 15000)
            print(f"simulate without a scan: longest decode {longest}", flush=True)
            tel = torch.full((C,), -9, dtype=torch.int64, device="cuda:0")
            comp = torch.full((C, n), -9, dtype=torch.int32, device="cuda:0")
            call = lambda: ctx.simulate(_dev(rows), _dev(s), _dev(o), M, tel_out=tel, completion_out=comp)
            if longest > 16384:
                with pytest.raises(kvsched.KvschedError) as e:
                    call()
                torch.cuda.synchronize()
                assert e.value.code == -2 and (tel == -9).all() and (comp == -9).all()
                continue
            call()
            assert ctx.device_status() == (kvsched.DEV_BAD_ORDER if longest == 15000 else 0)
            good = [c for c in range(C) if longest != 15000 or c != C // 2]
            tel_o, comp_o = oracle.simulate_many(s, o, M, rows[good], literal=False)
            assert (tel.cpu().numpy()[good] == tel_o).all() and (comp.cpu().numpy()[good] == comp_o).all()
    finally:
        ctx.close()


def test_status_behind_a_launch_that_fails():
    """A grid of 2^32 lanes is more than a launch takes.  Whatever the call gives, the next one's status is its own, not that of the
    call before the one that failed."""
    import torch
    from paper_2508_06133_amd import kvsched

    n, C = 33, 1 << 26  # (the buffers are there in full: a launch that is taken after all stays within them)
    rng = np.random.default_rng(5)
    s, o = _dev(rng.integers(1, 50, n)), _dev(rng.integers(1, 30, n))
    good, faulty = _dev(_rows(rng, n, 6, False)), _dev(_rows(rng, n, 6, True))
    many = torch.zeros((C, n), dtype=torch.int32, device="cuda:0")
    tel = torch.empty(C, dtype=torch.int64, device="cuda:0")
    ctx = kvsched.Context(0)
    try:
        ctx.set_o_max(30)
        for between in range(2):
            ctx.simulate(faulty, s, o, 400)
            assert ctx.device_status() == kvsched.DEV_BAD_ORDER
            print(f"simulate without a scan: {C} rows of {n}", flush=True)
            try:
                ctx.simulate(many, s, o, 400, completions=False, tel_out=tel)
                torch.cuda.synchronize()
            except kvsched.KvschedError as e:
                assert e.code == -3
            ctx.simulate(good, s, o, 400)
            assert ctx.device_status() == 0
            if between == 0:
                ctx.simulate(good, s, o, 400)
    finally:
        ctx.close()


@pytest.mark.parametrize("n,C", [(8, 70), (40, 20), (256, 6)])
def test_status_of_faulty_rows_after_a_wrong_guess(n, C):
    """Decodes longer than the register file of the call before: the first launch leaves everything but the status words as it is, and the
    second reports faulty rows where that one has said the status is.  Then a good call, whose guess is right."""
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    ctx = kvsched.Context(0)
    try:
        for longest in (40, 600, 3000, 5000, 9000, 40, 3000, 14336, 40, 9000):
            s, o = rng.integers(1, 50, n).astype(np.int32), rng.integers(1, 30, n).astype(np.int32)
            o[n // 2] = longest
            for faulty in (True, False, False):
                rows = _rows(rng, n, C, faulty)
                print(f"simulate without a scan: n={n} C={C} longest decode {longest} faulty={faulty}", flush=True)
                tel, comp = ctx.simulate(_dev(rows), _dev(s), _dev(o), 18000)
                assert ctx.device_status() == (kvsched.DEV_BAD_ORDER if faulty else 0)
                good = [c for c in range(C) if not faulty or c != C // 2][:8]
                tel_o, comp_o = oracle.simulate_many(s, o, 18000, rows[good], literal=False)
                tel, comp = tel.cpu().numpy(), comp.cpu().numpy()
                assert (tel[good] == tel_o).all() and (comp[good] == comp_o).all()
                assert (tel == -1).sum() == (1 if faulty else 0)
    finally:
        ctx.close()


@pytest.mark.parametrize("n,C", [(8, 70), (40, 20)])
def test_status_of_replays(n, C):
    """A captured call has its scan ahead: every replay leaves its own status, between eager calls that have none ahead."""
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    s, o = rng.integers(1, 50, n).astype(np.int32), rng.integers(1, 30, n).astype(np.int32)
    ds, do, M = _dev(s), _dev(o), 300
    rows = _dev(_rows(rng, n, C, False))
    tel = torch.empty(C, dtype=torch.int64, device="cuda:0")
    comp = torch.empty((C, n), dtype=torch.int32, device="cuda:0")
    ctx = kvsched.Context(0)
    try:
        ctx.set_o_max(30)
        ctx.simulate(rows, ds, do, M, tel_out=tel, completion_out=comp)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ctx.simulate(rows, ds, do, M, tel_out=tel, completion_out=comp)
        for turn, faulty in enumerate((True, False, False, True, True, False)):
            if turn % 2:
                ctx.simulate(_dev(_rows(rng, n, C, turn == 3)), ds, do, M)
                assert ctx.device_status() == (kvsched.DEV_BAD_ORDER if turn == 3 else 0)
            new = _rows(rng, n, C, faulty)
            rows.copy_(_dev(new))
            print(f"captured simulate: n={n} C={C} replay {turn} faulty={faulty}", flush=True)
            graph.replay()
            torch.cuda.synchronize()
            assert ctx.device_status() == (kvsched.DEV_BAD_ORDER if faulty else 0)
            good = [c for c in range(C) if not faulty or c != C // 2]
            tel_o, comp_o = oracle.simulate_many(s, o, M, new[good], literal=False)
            assert (tel.cpu().numpy()[good] == tel_o).all() and (comp.cpu().numpy()[good] == comp_o).all()
    finally:
        ctx.close()
