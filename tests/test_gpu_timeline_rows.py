"""Timelines whose windows end at the rows where the register kernel's pieces of code change: the longest
window in one piece, the four rows with limits, the segments of the row offsets, the last row of each file."""
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


@pytest.mark.parametrize("o_max", [512, 2048, 4096, 8192, 14336])
@pytest.mark.parametrize("crowded", [2, 6, 40])
def test_rows_at_the_edges(ctx, o_max, crowded):
    import torch

    print(f"o_max={o_max} crowded={crowded}", flush=True)
    rng = np.random.default_rng(o_max + crowded)
    edges = [64 * r + d for r in (1, 2, 4, 5, 8, 9, 12, 13, 14, 32, 64, 65, 66, 67, 131, 132, 133, 197, 198, 199, 223)
             for d in (-1, 0, 1) if 1 <= 64 * r + d <= o_max]
    n = 260
    o = np.concatenate([[o_max], rng.choice(edges, n - 1)]).astype(np.int32)
    s = rng.integers(1, 600, n).astype(np.int32)
    M = int((s + o).max()) + crowded * 700  # few at once: requests wait, the window moves over many rows
    orders = np.stack([rng.permutation(n) for _ in range(6)]).astype(np.int32)
    ctx.set_o_max(o_max)
    tel, comp = ctx.simulate(torch.from_numpy(orders).cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(o).cuda(), M)
    for row in range(len(orders)):
        _, want, total = oracle.simulate(s, o, M, orders[row], literal=False)[:3]
        assert int(tel[row].item()) == total
        assert (comp[row].cpu().numpy() == np.asarray(want)).all()
    assert ctx.device_status() == 0


def test_lengths_that_change_from_call_to_call(ctx):
    """No bound from the caller: a call may meet longer decodes than the one before, or shorter ones."""
    import torch

    ctx.set_o_max(0)
    rng = np.random.default_rng(9)
    n = 70
    for o_max in (300, 300, 5000, 200, 14000, 16384, 16384, 40, 2048, 2049, 2048):
        print(f"o_max={o_max}", flush=True)
        o = rng.integers(1, o_max + 1, n).astype(np.int32)
        o[11] = o_max
        s = rng.integers(1, 400, n).astype(np.int32)
        M = int((s + o).max()) + 900
        orders = np.stack([rng.permutation(n) for _ in range(3)]).astype(np.int32)
        tel, comp = ctx.simulate(torch.from_numpy(orders).cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(o).cuda(), M)
        for row in range(len(orders)):
            _, want, total = oracle.simulate(s, o, M, orders[row], literal=False)[:3]
            assert int(tel[row].item()) == total
            assert (comp[row].cpu().numpy() == np.asarray(want)).all()
        assert ctx.device_status() == 0


@pytest.mark.parametrize("o_max", [2048, 4096, 8192, 14336])
@pytest.mark.parametrize("crowded", [1, 12])
def test_rows_where_a_request_no_longer_is_one_piece(ctx, o_max, crowded):
    """Windows of 12 to 14, 28 to 30, 35 to 38 and 63 to 66 rows, as far as the file has them, from every place in a row
    (short requests in between move the round on by a little)."""
    import torch

    print(f"o_max={o_max} crowded={crowded}", flush=True)
    rng = np.random.default_rng(7 * o_max + crowded)
    edges = [64 * r + d for r in (11, 12, 13, 14, 27, 28, 29, 30, 34, 35, 36, 37, 38, 62, 63, 64, 65, 66)
             for d in (0, 1, 20, 63) if 64 * r + d <= o_max]
    n = 300
    o = np.where(rng.random(n) < 0.3, rng.integers(1, 90, n), rng.choice(edges, n)).astype(np.int32)
    o[rng.integers(0, n)] = o_max
    s = rng.integers(1, 300, n).astype(np.int32)
    M = int((s + o).max()) + crowded * 900
    orders = np.stack([rng.permutation(n) for _ in range(8)]).astype(np.int32)
    ctx.set_o_max(o_max)
    tel, comp = ctx.simulate(torch.from_numpy(orders).cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(o).cuda(), M)
    for row in range(len(orders)):
        _, want, total = oracle.simulate(s, o, M, orders[row], literal=False)[:3]
        assert int(tel[row].item()) == total
        assert (comp[row].cpu().numpy() == np.asarray(want)).all()
    assert ctx.device_status() == 0
