"""Local Swap Search where its splits change: the places of one wavefront and of the workgroup, the largest
backlog held in LDS, sizes beyond the table, values that are no lengths."""
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


def _lengths(n, smax, seed):
    rng = np.random.default_rng(seed)
    s = np.clip(np.rint(rng.lognormal(np.log(128.0), 0.8, n)), 4, smax).astype(np.int32)
    o = np.clip(np.rint(rng.lognormal(np.log(200.0), 0.9, n)), 1, 2048).astype(np.int32)
    return s, o


@pytest.mark.parametrize("n,M,alpha", [
    (255, 60000, (0, 1)), (257, 60000, (5, 1)),        # one wavefront: 4 places per lane and more
    (511, 120000, (0, 1)), (513, 110000, (13, 1000)),
    (1023, 230000, (0, 1)), (1025, 260000, (5, 1)),    # up to here one wavefront, then the workgroup
    (2049, 500000, (0, 1)), (4097, 900000, (1, 1)),
    (6000, 1700000, (0, 1)), (8191, 500000, (5, 1)),   # the most that LDS holds
    (8192, 500000, (0, 1)),
    (3000, 1 << 23, (0, 1)),                           # one batch of everything
])
def test_splits(ctx, n, M, alpha):
    from paper_2508_06133_amd import kvsched
    import torch

    print(f"n={n} M={M} alpha={alpha}", flush=True)
    s, o = _lengths(n, 2048, n)
    ds, do = torch.from_numpy(s).cuda(), torch.from_numpy(o).cuda()
    if alpha == (0, 1):
        want = oracle.local_swap(s, o, M, True)
        order, ends, F, swaps, nb = ctx.local_swap(ds, do, M)
    else:
        want = oracle.local_swap(s, o, M, True, alpha=alpha)
        order, ends, F, swaps, nb = ctx.phase1_G(kvsched.SOLVER_LOCAL_SWAP, ds, do, M, alpha)
    k = int(nb.item())
    assert k == len(want[1])
    assert (order.cpu().numpy() == want[0]).all()
    assert (ends.cpu().numpy()[:k] == want[1]).all() and (ends.cpu().numpy()[k:] == 0).all()
    assert (swaps.cpu().numpy()[:k] == want[3]).all() and (swaps.cpu().numpy()[k:] == 0).all()
    assert np.allclose(F.cpu().numpy()[:k], want[2], rtol=1e-12, atol=0.0) and (F.cpu().numpy()[k:] == 0).all()
    assert ctx.device_status() == 0


@pytest.mark.parametrize("largest", [16383, 16384, 40000])
def test_sizes_about_the_table(ctx, largest):
    import torch

    print(f"largest={largest}", flush=True)
    s, o = _lengths(400, 1024, largest)
    s[7], o[7] = largest - 100, 100
    M = 100000
    want = oracle.local_swap(s, o, M, True)
    order, ends, F, swaps, nb = ctx.local_swap(torch.from_numpy(s).cuda(), torch.from_numpy(o).cuda(), M)
    assert int(nb.item()) == len(want[1])
    assert (order.cpu().numpy() == want[0]).all()
    assert (swaps.cpu().numpy()[: len(want[3])] == want[3]).all()
