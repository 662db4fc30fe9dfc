"""GPU parity with the CPU oracle where orders go to and fro between bursts of requests and requests one at a time, so that the number of
requests looked at one by one before the memory left is measured grows to its upper end and falls again: the files of 65 rows and
more, placed in full and resumed from another order's states, groups around the least that is added at once."""
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


def _phases(rng, n, o_max, burst):
    """Stretches of `burst` short requests behind each long one, of long ones alone, and of lengths all over."""
    s, o = rng.integers(1, 60, n), rng.integers(1, o_max + 1, n)
    k, kind = 0, 0
    while k < n:
        m = min(n - k, int(rng.integers(20, 90)))
        if kind % 3 == 0:
            o[k : k + m] = np.where(np.arange(m) % (burst + 1) == 0, o_max, rng.integers(1, 3, m))
        elif kind % 3 == 1:
            o[k : k + m] = o_max - rng.integers(0, 2, m)
        k, kind = k + m, kind + 1
    o[n // 2] = o_max
    return s.astype(np.int32), o.astype(np.int32)


@pytest.mark.parametrize("o_max", [2049, 4096, 8192, 14336])
@pytest.mark.parametrize("burst", [2, 3, 4, 5, 17])
def test_bursts_and_single_requests(ctx, o_max, burst):
    import torch

    n = 400
    rng = np.random.default_rng(o_max + burst)
    s, o = _phases(rng, n, o_max, burst)
    rows = np.tile(np.arange(n, dtype=np.int32), (8, 1))
    for r in rows[1:]:  # (near one another: some resume from the first one's states when they are many)
        for i, j in rng.integers(n // 2, n, (6, 2)):
            r[i], r[j] = r[j], r[i]
    rows[7] = rng.permutation(n)
    d = [torch.from_numpy(x).to("cuda:0") for x in (np.tile(rows, (130, 1)), s, o)]
    for share in (3, 12, 60):
        M = max(int((s + o).max()), int((s + o).sum()) // share)
        print(f"bursts and single requests: o_max={o_max} burst={burst} M={M}", flush=True)
        want = [oracle.simulate(s, o, M, r, literal=False)[1:] for r in rows]
        for C in (8, 1040):
            for least in (-1, 2):
                ctx.set_resume_min_rows(least)
                tel, comp = ctx.simulate(d[0][:C], d[1], d[2], M)
                tel, comp = tel.cpu().numpy(), comp.cpu().numpy()
                for c in (*range(8), *range(C - 8, C)):
                    assert tel[c] == want[c % 8][1] and (comp[c] == want[c % 8][0]).all(), (C, least, c)
        ctx.set_resume_min_rows(-1)
        assert ctx.device_status() == 0
