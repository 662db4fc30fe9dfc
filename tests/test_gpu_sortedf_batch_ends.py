"""GPU parity of kvsched_sortedF with the CPU oracle where the order within the batches reads their ends, a lane each and 64 at a
time: numbers of batches about 64 and its multiples, the last batch full and of one request."""
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


@pytest.mark.parametrize("feas", [0, 1])
@pytest.mark.parametrize("batches", [1, 2, 63, 64, 65, 66, 127, 128, 129, 255, 256, 257, 320])
def test_numbers_of_batches(ctx, batches, feas):
    import torch

    rng = np.random.default_rng(batches)
    for each, n_more in ((1200 // batches + 1, 0), (1200 // batches + 1, 1), (16384 // batches, 0)):
        n = min(each * batches + n_more, 16385)
        s, o = np.full(n, 2, dtype=np.int32), np.full(n, 3, dtype=np.int32)  # (`each` of them fill the budget)
        if feas == 0:
            o = rng.integers(1, 5, n).astype(np.int32)  # (the size the same, the decode length not)
            s = (5 - o).astype(np.int32)
            s[s == 0], o[s == 0] = 1, 4
        M = 5 * each
        print(f"sortedF batch ends: n={n} batches of {each}, feas={feas}", flush=True)
        order_o, ends_o, F_o = oracle.sortedF(s, o, M, 1, feas)
        order, ends, F, nb = ctx.sortedF(torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0"), M, 1, feas)
        k = int(nb.item())
        assert ctx.device_status() == 0
        assert k == len(ends_o) and (ends.cpu().numpy()[:k] == ends_o).all()
        assert (order.cpu().numpy() == order_o).all()
        assert np.allclose(F.cpu().numpy()[:k], F_o, rtol=1e-12, atol=0.0)
