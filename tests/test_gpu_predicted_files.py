"""GPU parity of kvsched_simulate_predicted with the CPU oracle at the edges of its register files (decode lengths and
estimates around 512, 1024, 2048, 4096 rounds), with estimates below and above the truth, and with more requests running
at once than the first launch's list holds."""
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


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda:0")


def _check(ctx, s, o, est, M, rows):
    tel, comp, ev = ctx.simulate_predicted(_dev(rows), _dev(s), _dev(o), _dev(est), M)
    assert ctx.device_status() == 0
    tel, comp, ev = tel.cpu().numpy(), comp.cpu().numpy(), ev.cpu().numpy()
    for c in range(rows.shape[0]):
        _, c_o, tel_o, ev_o, _ = oracle.simulate_predicted(s, o, est if est.ndim == 1 else est[c], M, rows[c])
        assert tel[c] == tel_o and (comp[c] == c_o).all() and ev[c] == int(ev_o.sum()), c
    return int(ev.sum())


@pytest.mark.parametrize("o_max", [63, 64, 511, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
def test_register_files(ctx, o_max):
    inst = workloads.tight_instance(o_max, 140, o_max)
    rng = np.random.default_rng(o_max)
    rows = np.stack([rng.permutation(inst.n) for _ in range(12)]).astype(np.int32)
    lower, upper = workloads.prediction_intervals(o_max, inst.s, inst.o, inst.M, 0.4)
    upper = np.minimum(upper, max(o_max, int(inst.o.max()))).astype(np.int32)
    mixed = np.where(rng.random((12, inst.n)) < 0.5, lower, upper).astype(np.int32)
    for what, est in (("lower", lower), ("upper", upper), ("exact", inst.o), ("one per row", mixed)):
        print(f"predicted, register files: o_max={o_max} M={inst.M} {what}", flush=True)
        _check(ctx, inst.s, inst.o, est, inst.M, rows)


@pytest.mark.parametrize("n", [1000, 1300, 2500])
def test_more_running_requests_than_the_first_launch_holds(ctx, n):
    rng = np.random.default_rng(n)
    s, o = np.ones(n, dtype=np.int32), rng.integers(1, 1900, n).astype(np.int32)
    lower = np.maximum(1, o // 2).astype(np.int32)
    rows = np.stack([rng.permutation(n) for _ in range(3)]).astype(np.int32)
    for M in (int(0.4 * n * 950), 5000000):
        print(f"predicted, long lists: n={n} M={M}", flush=True)
        _check(ctx, s, o, lower, M, rows)


def test_many_requests_that_finish_together(ctx):
    n = 600
    s, o = np.full(n, 2, dtype=np.int32), np.full(n, 40, dtype=np.int32)
    o[::7] = 41
    rows = np.stack([np.arange(n), np.arange(n)[::-1]]).astype(np.int32)
    for est in (o, np.full(n, 40, dtype=np.int32), np.full(n, 11, dtype=np.int32), np.full(n, 60, dtype=np.int32)):
        for M in (300 * 42, 130 * 42, 3000):
            print(f"predicted, finishing together: M={M} est {int(est[0])}", flush=True)
            _check(ctx, s, o, est.astype(np.int32), M, rows)


@pytest.mark.parametrize("o_max", [5000, 8192, 16384])
def test_rings(ctx, o_max):
    """Beyond 4096 rounds: the projection as a ring; requests that run out together among long ones."""
    inst = workloads.tight_instance(o_max, 50, o_max)
    rng = np.random.default_rng(o_max)
    s = np.concatenate([inst.s, np.full(40, 2, dtype=np.int32)]).astype(np.int32)
    o = np.concatenate([inst.o, np.full(40, 40, dtype=np.int32)]).astype(np.int32)
    o[0] = o_max
    rows = np.stack([rng.permutation(len(o)) for _ in range(1 if o_max > 8192 else 3)]).astype(np.int32)
    M = max(inst.M, int((s + o).max()))
    lower, upper = workloads.prediction_intervals(o_max, s, o, M, 0.4)
    upper = np.minimum(upper, 16384).astype(np.int32)
    for what, est in (("lower", lower), ("upper", upper), ("exact", o)):
        print(f"predicted, rings: o_max={o_max} M={M} {what}", flush=True)
        _check(ctx, s, o, est, M, rows)


@pytest.mark.parametrize("n", [1000, 1100, 1300])
def test_long_lists_with_the_largest_register_file(ctx, n):
    rng = np.random.default_rng(n)
    s, o = np.ones(n, dtype=np.int32), rng.integers(1, 4001, n).astype(np.int32)
    o[5] = 4000
    lower = np.maximum(1, o // 2).astype(np.int32)
    rows = rng.permutation(n)[None].astype(np.int32)
    for M in (int(0.4 * n * 2000), 9000000):
        print(f"predicted, long lists: n={n} M={M}", flush=True)
        _check(ctx, s, o, lower, M, rows)
