"""GPU parity of kvsched_online with the CPU oracle where its small variants end: windows around the 64 places of
one row of registers and the 128 of two, and decode lengths around the 256 rounds that an admission keeps from its
test."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waiting", [1, 2, 63, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("longest", [1, 64, 255, 256, 257, 512, 513, 1100])
def test_windows_and_lengths(waiting, longest):
    import torch
    from paper_2508_06133_amd import kvsched

    rng = np.random.default_rng(1000 * waiting + longest)
    n = waiting + 40
    a = np.concatenate([np.zeros(waiting), np.sort(rng.integers(0, 2 * longest + 40, 40))]).astype(np.int32)
    s = rng.integers(1, 200, n).astype(np.int32)
    o = np.where(rng.random(n) < 0.3, longest, rng.integers(1, longest + 1, n)).astype(np.int32)
    M = int((s + o).max()) + 3 * longest + 500
    cases = [(3, 10, 300, (1, 2)), (3, 1, 64, (0, 1)), (1, 1, 0, (0, 0)), (0, 1, 0, (0, 0))]
    desc = np.array([[0, n, *c[:3], *c[3], k * n] for k, c in enumerate(cases)], dtype=np.int32)
    print(f"online: {waiting} waiting, decodes up to {longest}, M={M}", flush=True)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    ctx = kvsched.Context(0)
    try:
        comp, stats = ctx.online(dev(desc), dev(a), dev(s), dev(o), M,
                                 torch.full((len(cases) * n,), -7, dtype=torch.int32, device="cuda:0"), backlog_cap=512)
        assert ctx.device_status() == 0
        for k, c in enumerate(cases):
            _, c_o, st_o = oracle.online(a, s, o, M, *c)
            assert tuple(int(x) for x in stats[k]) == st_o, c
            assert (comp[k * n : (k + 1) * n].cpu().numpy() == c_o).all(), c
    finally:
        ctx.close()
