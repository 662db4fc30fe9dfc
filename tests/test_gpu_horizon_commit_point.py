"""The commit point of a horizon step, the k-th completion and what has been admitted and has completed by it: rounds beyond 2^20, many
completions in one round, numbers of requests around what a workgroup holds in registers, the first and the last completion."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lengths(kind, n, rng):
    if kind == "late":     # hardly two at a time: completions up to some millions of rounds
        return rng.integers(1, 200, n), rng.integers(1000, 2048, n), 2600
    if kind == "together":  # all at once, three different rounds
        return np.full(n, 3), rng.choice([5, 6, 300], n), (1 << 30) - 1
    return rng.integers(1, 300, n), rng.integers(1, 400, n), 40000


@pytest.mark.parametrize("kind", ["late", "together", "mixed"])
@pytest.mark.parametrize("n", [1, 63, 1023, 1025, 4097, 16384, 16386])
def test_commit_point(kind, n):
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    s, o, M = _lengths(kind, n, rng)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to("cuda:0")
    ds, do = dev(s), dev(o)
    ctx = kvsched.Context(0)
    try:
        for every in sorted({1, max(1, n // 3), n, n + 7}):
            print(f"commit point: {kind} n={n} every={every}", flush=True)
            order = dev(rng.permutation(n))
            moves = dev(np.array([[0, n - 1, n - 1], [0, n // 2, n - 1]]))
            _, res = ctx.horizon_step(order, moves, ds, do, M, 0, every)
            _, _, _, committed, completed, T = (int(x) for x in res.cpu().numpy())
            assert ctx.device_status() == 0
            _, comp = ctx.simulate(order[None, :], ds, do, M)[:2]
            ends = comp[0].cpu().numpy().astype(np.int64)
            starts = ends - o
            want = int(np.sort(ends)[min(every, n) - 1])
            assert T == want and completed == int((ends <= want).sum()) and committed == int((starts <= want).sum())
            assert kind != "late" or every < n or n < 1023 or T > 1 << 19
    finally:
        ctx.close()


@pytest.mark.parametrize("states", [True, False])
@pytest.mark.parametrize("n", [1, 5, 100, 128, 1500])
def test_faulty_order(n, states):
    """An order that is no permutation: nothing is committed where no states are kept (up to 128 positions, or if the caller rules them out), whatever
    the completion rounds' buffer held; the numbers are the same in every call; and it is reported."""
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    s, o, M = _lengths("mixed", n, rng)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to("cuda:0")
    ds, do = dev(s), dev(o)
    moves = dev(np.array([[0, n - 1, n - 1], [0, 0, n - 1]]))
    ctx = kvsched.Context(0)
    try:
        if not states:
            ctx.set_resume_min_rows(0)
        for at, wrong in ((n - 1, -1), (0, n), (n // 2, 2**31 - 1), (n - 1, "again")):
            faulty = rng.permutation(n)
            if wrong == "again":
                if n == 1:
                    continue
                wrong = faulty[0]
            faulty[at] = wrong
            for every in sorted({1, max(1, n // 3), n}):
                seen = []
                for left in (-1, 0, 2**30, 77):  # what the completion rounds' buffer holds before
                    print(f"commit point, faulty order: n={n} states={states} id {wrong} at {at} every={every} left={left}", flush=True)
                    comp = torch.full((n,), left, dtype=torch.int32, device="cuda:0")
                    _, res = ctx.horizon_step(dev(faulty), moves, ds, do, M, 0, every, completion_out=None if left == 77 else comp)
                    assert ctx.device_status() == kvsched.DEV_BAD_ORDER
                    seen.append(tuple(int(x) for x in res.cpu().numpy()))
                assert len(set(seen[:3])) == 1 and seen[0][0] == -1 and seen[0][2] == -1
                if n <= 128 or not states:
                    assert seen[0] == seen[3] and seen[0][3:] == (0, 0, 0)
        order = rng.permutation(n)  # and a good one afterwards
        _, res = ctx.horizon_step(dev(order), moves, ds, do, M, 0, n)
        assert ctx.device_status() == 0 and [int(x) for x in res.cpu().numpy()][3:5] == [n, n]
    finally:
        ctx.close()
