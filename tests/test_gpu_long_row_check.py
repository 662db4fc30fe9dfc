"""Long orders that are no permutations are found, and only those: sizes around whole words of the bitmap and the stretch
a workgroup reads at once, numbers of rows on both sides of the line between its two sizes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows", [(16384, 6), (16385, 513), (16415, 512), (18431, 520), (20481, 2), (40000, 515)])
def test_rows(n, rows):
    import torch
    from paper_2508_06133_amd import kvsched

    gen = torch.Generator(device="cuda:0").manual_seed(n)
    orders = torch.argsort(torch.rand((rows, n), device="cuda:0", generator=gen), dim=1).to(torch.int32).contiguous()
    s = torch.ones(n, dtype=torch.int32, device="cuda:0")
    ctx = kvsched.Context(0)
    try:
        ctx.set_o_max(64)
        print(f"long rows: n={n} rows={rows}", flush=True)
        good, _ = ctx.simulate(orders, s, s, 4 * n, completions=False)
        assert ctx.device_status() == 0 and bool((good == n).all())  # (all start in round 0 and last one round)
        for at, value in ((0, -1), (n - 1, n), (n // 2, 2**31 - 1), (n - 1, int(orders[rows // 2, 0])), (0, int(orders[rows // 2, n - 1]))):
            bad = orders.clone()
            bad[rows // 2, at] = value
            tel, _ = ctx.simulate(bad, s, s, 4 * n, completions=False)
            assert ctx.device_status() == kvsched.DEV_BAD_ORDER
            assert np.flatnonzero(tel.cpu().numpy() != n).tolist() == [rows // 2] and int(tel[rows // 2]) == -1
    finally:
        ctx.close()
