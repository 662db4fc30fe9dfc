"""GPU parity with the CPU oracle where memory is counted in numbers that just fit in 32 bits: M = 2^30 - 1 and prompts of 2^28 and
2^29 tokens that leave the last few hundred tokens of it to the decodes."""
import numpy as np
import pytest

import oracle

M = 2**30 - 1


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda:0")


def _instance(rng, n, longest):
    """Two or four requests share the budget: what is left of it beside their prompts is about what their decodes take."""
    o = rng.integers(1, 300, n).astype(np.int32)
    o[:: max(n // 3, 1)] = longest
    half = rng.random(n) < 0.3
    s = np.where(half, 2**29, 2**28) - rng.integers(1, 250, n)
    s = np.minimum(s, M - o - 1).astype(np.int32)
    s[rng.random(n) < 0.1] = 1
    return s, o


def _rows(rng, n, count):
    return np.argsort(rng.random((count, n)), axis=1).astype(np.int32)


# (longest decode: register files of 9, 33 and 65 rows, the ring)
@pytest.mark.gpu
@pytest.mark.parametrize("n,longest", [(60, 300), (60, 1500), (200, 400), (40, 4000), (60, 5000), (40, 16000)])
def test_predicted(n, longest):
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n + longest)
    s, o = _instance(rng, n, longest)
    rows = _rows(rng, n, 6 if longest < 10000 else 2)
    lower = np.array([rng.integers(1, x + 1) for x in o], dtype=np.int32)
    upper = np.minimum(np.array([rng.integers(x, x + 200) for x in o]), np.minimum(M - s, 16384)).astype(np.int32)
    ctx = kvsched.Context(0)
    evictions = 0
    try:
        for what, est in (("lower", lower), ("upper", upper), ("either", np.where(rng.random(n) < 0.5, lower, upper).astype(np.int32))):
            print(f"predicted, largest numbers: n={n} longest={longest} {what}", flush=True)
            tel, comp, ev = (x.cpu().numpy() for x in ctx.simulate_predicted(_dev(rows), _dev(s), _dev(o), _dev(est), M))
            assert ctx.device_status() == 0
            for c in range(len(rows)):
                _, c_o, tel_o, ev_o, _ = oracle.simulate_predicted(s, o, est, M, rows[c])
                assert tel[c] == tel_o and (comp[c] == c_o).all() and ev[c] == int(ev_o.sum()), (what, c)
                evictions += int(ev_o.sum())
        assert evictions > 0
    finally:
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n,rows", [(1, 3), (8, 130), (16, 8192), (32, 16384), (40, 20)])
def test_short_rows(n, rows):
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(n)
    orders = _rows(rng, n, rows)
    some = np.r_[0:min(rows, 16), max(rows - 16, 0):rows]
    ctx = kvsched.Context(0)
    try:
        for turn, longest in enumerate((300, 300, 5000, 14000)):
            s, o = _instance(rng, n, longest)
            print(f"short rows, largest numbers: n={n} rows={rows} longest={longest} turn={turn}", flush=True)
            tel, comp = ctx.simulate(_dev(orders), _dev(s), _dev(o), M)
            assert ctx.device_status() == 0
            tel_o, comp_o = oracle.simulate_many(s, o, M, orders[some])
            assert (tel.cpu().numpy()[some] == tel_o).all() and (comp.cpu().numpy()[some] == comp_o).all()
    finally:
        ctx.close()
