"""kvsched_exact_dp against all subsets of the remaining requests, where single requests hold more than 2^24 tokens: loads that
differ by a token or two, the later requests the lighter, and budgets that the lightest of them fill exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _phase1(s, o, M, tie, alpha=(0, 1)):
    """(order, batch ends, F) with every batch the best subset: least F, then the size, then the least load, then the set
    whose latest request is the earliest, then whose second latest is (the least as a binary number)."""
    left, order, ends, F = list(range(len(s))), [], [], []
    while left:
        w = np.zeros(1, dtype=np.int64)
        v, k = w.copy(), w.copy()
        for i in left:  # bit b of a subset's number: the b-th of those left
            w, v, k = np.concatenate([w, w + s[i] + o[i]]), np.concatenate([v, v + alpha[0] * s[i] + alpha[1] * o[i]]), np.concatenate([k, k + 1])
        ok = np.flatnonzero((w <= M) & (k > 0))
        best = None
        for size in np.unique(k[ok]):
            of_size = ok[k[ok] == size]
            least = of_size[v[of_size] == v[of_size].min()]
            at = least[np.argmin(w[least])]  # (the first of equal ones)
            size, value = int(size), int(v[at])
            d = 0 if best is None else value * best[0] ** 2 - best[1] * size ** 2
            if best is None or d < 0 or (d == 0 and tie == 0):
                best = (size, value, int(at))
        members = [i for b, i in enumerate(left) if best[2] >> b & 1]
        order += sorted(members, key=lambda i: (o[i], i))
        ends.append(len(order))
        F.append(best[1] / (alpha[1] * best[0] ** 2))
        left = [i for i in left if i not in members]
    return order, ends, F


def _near_ties(rng, n, largest):
    """n requests, of which some are within a few tokens of largest / k, the later the lighter; M is what the lightest k hold."""
    o = rng.integers(200, 3000, n)
    k = int(rng.integers(3, n - 2))
    near = int(rng.integers(k + 1, n))
    load = np.concatenate([rng.integers(largest // 2, largest, n - near), np.sort(-(-largest // k) + rng.integers(0, 5, near))[::-1]])
    load[0] = largest
    return (load - o).astype(np.int32), o.astype(np.int32), int(np.sort(load)[:k].sum())


def _check(ctx, s, o, M, alpha=(0, 1)):
    import torch
    from paper_2508_06133_amd import kvsched

    ds, do = torch.from_numpy(s).to("cuda:0"), torch.from_numpy(o).to("cuda:0")
    s, o = s.astype(np.int64), o.astype(np.int64)
    for tie in (0, 1):
        order_r, ends_r, F_r = _phase1(s, o, M, tie, alpha)
        if alpha[0]:
            order, ends, F, _, nb = ctx.phase1_G(kvsched.SOLVER_EXACT_DP, ds, do, M, alpha, tie, 0)
        else:
            order, ends, F, nb = ctx.exact_dp(ds, do, M, 0, tie)
        k = int(nb.item())
        assert ctx.device_status() == 0 and k == len(ends_r)
        assert ends.cpu().numpy()[:k].tolist() == ends_r and order.cpu().numpy().tolist() == order_r
        assert np.allclose(F.cpu().numpy()[:k], F_r, rtol=1e-12, atol=0.0)


@pytest.fixture(scope="module")
def ctx():
    from paper_2508_06133_amd import kvsched

    c = kvsched.Context(0)
    yield c
    c.close()


def test_seven_of_twelve(ctx):
    """Seven requests fit, of nearly equal loads about M / 7 (F = 203.2), where the best six have F = 207.9."""
    s = [4678167, 3586973, 4678529, 4431044, 3976920, 4594924, 4301280, 4440085, 25541260, 23954647, 14463658, 29991751]
    o = [1478, 815, 1115, 1581, 1978, 1522, 973, 1974, 776, 2020, 866, 454]
    print("exact_dp, wide loads: seven of twelve", flush=True)
    _check(ctx, np.array(s, dtype=np.int32), np.array(o, dtype=np.int32), 30019713)


@pytest.mark.parametrize("largest", [16770000, 16777300, 29999999, 60000000])
@pytest.mark.parametrize("n", [8, 11, 12, 16])
def test_near_ties(ctx, n, largest):
    rng = np.random.default_rng(n + largest)
    for case in range(4):
        s, o, M = _near_ties(rng, n, largest)
        print(f"exact_dp, wide loads: n={n} largest={largest} case={case} M={M}", flush=True)
        _check(ctx, s, o, M)


@pytest.mark.parametrize("alpha", [(1, 1), (1, 50), (7, 2)])
def test_near_ties_weighted(ctx, alpha):
    """Values above 2^24 as well as loads."""
    rng = np.random.default_rng(alpha[0] + alpha[1])
    for n in (11, 14):
        s, o, M = _near_ties(rng, n, 20999999)
        print(f"exact_dp, wide loads: n={n} M={M} alpha={alpha}", flush=True)
        _check(ctx, s, o, M, alpha)
