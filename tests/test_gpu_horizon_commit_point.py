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
