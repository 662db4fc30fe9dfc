"""GPU parity of kvsched_exact_dp's many-workgroup variant with the CPU oracle: numbers of requests around the four
that a launch takes, row lengths around its tiles, both constraints, both tie rules, and the G metric (whose bound on the
batch size is looser)."""
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


def _dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda:0")


@pytest.mark.parametrize("feas", [0, 1])
@pytest.mark.parametrize("n,smax,omax,M", [(1, 900, 900, 9000), (2, 60, 60, 9000), (3, 60, 60, 8191), (4, 90, 90, 8192),
                                           (5, 90, 90, 8703), (66, 70, 70, 8704), (67, 300, 90, 9215), (121, 90, 200, 9216),
                                           (150, 2, 2, 20000)])
def test_sizes(ctx, n, smax, omax, M, feas):
    rng = np.random.default_rng(n)
    s, o = rng.integers(1, smax + 1, n).astype(np.int32), rng.integers(1, omax + 1, n).astype(np.int32)
    for tie in (0, 1):
        print(f"exact_dp large: n={n} M={M} feas={feas} tie={tie}", flush=True)
        order_o, ends_o, F_o = oracle.exact_phase1(s, o, M, feas, tie)
        order, ends, F, nb = ctx.exact_dp(_dev(s), _dev(o), M, feas, tie)
        k = int(nb.item())
        assert ctx.device_status() == 0 and k == len(ends_o)
        assert (ends.cpu().numpy()[:k] == ends_o).all() and (order.cpu().numpy() == order_o).all()
        assert np.allclose(F.cpu().numpy()[:k], F_o, rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("feas", [0, 1])
@pytest.mark.parametrize("alpha", [(0, 3), (1, 1), (7, 2)])
def test_g_metric(ctx, alpha, feas):
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(5)
    s, o = rng.integers(1, 400, 60).astype(np.int32), rng.integers(1, 400, 60).astype(np.int32)
    M = 8500
    print(f"exact_dp large, G metric {alpha} feas={feas}", flush=True)
    order_o, ends_o, G_o = oracle.exact_phase1(s, o, M, feas, 0, alpha)
    order, ends, G, _, nb = ctx.phase1_G(kvsched.SOLVER_EXACT_DP, _dev(s), _dev(o), M, alpha, 0, feas)
    k = int(nb.item())
    assert ctx.device_status() == 0 and k == len(ends_o)
    assert (ends.cpu().numpy()[:k] == ends_o).all() and (order.cpu().numpy() == order_o).all()
    assert np.allclose(G.cpu().numpy()[:k], G_o, rtol=1e-12, atol=0.0)


@pytest.mark.parametrize("n,M", [(4, 1 << 29), (20, 1 << 28)])
def test_largest_tables(ctx, n, M):
    """Tables just within the documented 16 GiB.  Batches are known without the oracle: up to k_max = 1 / 3 of any of the
    requests share a batch, decodes are distinct and within a factor of two, so every batch is the k_max shortest that
    are left (F = 1/9 of their sum is below any pair's and any single one's)."""
    rng = np.random.default_rng(n)
    k_max = 1 if n == 4 else 3
    o = (4000 + rng.permutation(n) * 7).astype(np.int32)
    s = (M // (k_max + 1) + 1 + rng.integers(0, 5000, n)).astype(np.int32)
    assert (k_max + 1) * int((s + o).min()) > M and k_max * int((s + o).max()) <= M
    assert 2 * (k_max + 1) * (M + 1) * (4 + n / 16) <= 16 << 30
    print(f"exact_dp largest tables: n={n} M={M} k_max={k_max}", flush=True)
    order, ends, F, nb = ctx.exact_dp(_dev(s), _dev(o), M)
    k = int(nb.item())
    want_ends = np.minimum(np.arange(k_max, n + k_max, k_max), n)
    assert ctx.device_status() == 0 and k == len(want_ends)
    assert (order.cpu().numpy() == np.argsort(o)).all() and (ends.cpu().numpy()[:k] == want_ends).all()
    by_o = np.sort(o).astype(float)
    want_F = [by_o[a:b].sum() / (b - a) ** 2 for a, b in zip(np.r_[0, want_ends[:-1]], want_ends)]
    assert np.allclose(F.cpu().numpy()[:k], want_F, rtol=1e-12, atol=0.0)
