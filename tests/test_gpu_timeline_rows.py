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


@pytest.mark.parametrize("n", [70, 300])
@pytest.mark.parametrize("completions", [True, False])
def test_a_call_that_starts_with_the_last_calls_register_file(ctx, n, completions):
    """No bound from the caller, after a call with short decodes: too long a decode leaves the outputs as they are, a longer
    one than that file takes gives the right results, a faulty row among them is found."""
    import torch

    from paper_2508_06133_amd import kvsched

    print(f"n={n} completions={completions}", flush=True)
    rng = np.random.default_rng(n)
    ctx.set_o_max(0)
    s = rng.integers(1, 300, n).astype(np.int32)
    orders = np.stack([rng.permutation(n) for _ in range(5)]).astype(np.int32)

    def call(orders, o, M):
        tel = torch.full((5,), -7, dtype=torch.int64, device="cuda:0")
        comp = torch.full((5, n), -7, dtype=torch.int32, device="cuda:0")
        try:
            ctx.simulate(torch.from_numpy(orders).cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(o).cuda(), M,
                         completions, tel_out=tel, completion_out=comp)
            code = 0
        except kvsched.KvschedError as e:
            code = e.code
        torch.cuda.synchronize()
        return code, tel.cpu().numpy(), comp.cpu().numpy()

    for o_max in (100, 5000, 14000, 100):
        o = rng.integers(1, o_max + 1, n).astype(np.int32)
        o[3] = o_max
        short = np.minimum(o, 200)
        assert call(orders, short, 4000)[0] == 0
        long = o.copy()
        long[5] = 20000
        code, tel, comp = call(orders, long, 40000)
        assert code == -2 and (tel == -7).all() and (comp == -7).all()
        assert call(orders, short, 4000)[0] == 0
        faulty = orders.copy()
        faulty[2, 1] = faulty[2, 0]
        code, tel, comp = call(faulty, o, 16000)
        assert code == 0 and ctx.device_status() == kvsched.DEV_BAD_ORDER and tel[2] == -1
        for row in (0, 1, 3, 4):
            _, want, total = oracle.simulate(s, o, 16000, orders[row], literal=False)[:3]
            assert tel[row] == total
            assert not completions or (comp[row] == np.asarray(want)).all()
    # as many positions as a round counter cannot count: refused before anything is written
    m = 65600
    assert call(orders, short, 4000)[0] == 0
    o = np.full(m, 16384, np.int32)
    tel = torch.full((1,), -7, dtype=torch.int64, device="cuda:0")
    with pytest.raises(kvsched.KvschedError) as e:
        ctx.simulate(torch.arange(m, dtype=torch.int32, device="cuda:0")[None], torch.ones(m, dtype=torch.int32, device="cuda:0"),
                     torch.from_numpy(o).cuda(), 1 << 20, False, tel_out=tel)
    torch.cuda.synchronize()
    assert e.value.code == -2 and int(tel.item()) == -7
