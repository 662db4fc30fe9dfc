"""The native calls of a planning step give what the Python path gives, refuse what it refuses, and leave to it what is not a
plain tensor."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


class _Declined:
    """Stands for the native module and takes no call."""

    def __getattr__(self, name):
        return lambda *a: None


def _instance(n, C):
    import torch

    rng = np.random.default_rng(n)
    s, o = rng.integers(1, 60, n).astype(np.int32), rng.integers(1, 90, n).astype(np.int32)
    rows = np.stack([rng.permutation(n) for _ in range(C)]).astype(np.int32)
    return s, o, rows, [torch.from_numpy(x).to("cuda:0") for x in (s, o, rows)]


@pytest.mark.parametrize("n,C", [(1, 1), (7, 3), (61, 1), (300, 40), (1500, 2)])
def test_both_paths(monkeypatch, n, C):
    import torch
    from paper_2508_06133_amd import kvsched

    s_h, o_h, rows_h, (s, o, rows) = _instance(n, C)
    M = 900
    ctx = kvsched.Context(0)
    print(f"host calls: n={n} C={C}", flush=True)
    native = [*ctx.sortedF(s, o, M, kvsched.TIE_SMALLER, kvsched.FEAS_PROFILE), *ctx.simulate(rows, s, o, M)]
    native.append(ctx.argmin(native[4]))
    assert ctx.simulate(rows, s, o, M, completions=False)[1] is None
    order_o, ends_o, _ = oracle.sortedF(s_h, o_h, M, kvsched.TIE_SMALLER, kvsched.FEAS_PROFILE)
    tel_o, comp_o = oracle.simulate_many(s_h, o_h, M, rows_h)
    assert (native[0].cpu().numpy() == order_o).all() and (native[1].cpu().numpy()[: len(ends_o)] == ends_o).all()
    assert (native[4].cpu().numpy() == tel_o).all() and (native[5].cpu().numpy() == comp_o).all()
    assert native[6].tolist() == [int(tel_o.argmin()), int(tel_o.min())]
    monkeypatch.setattr(kvsched, "_host", _Declined())
    python = [*ctx.sortedF(s, o, M, kvsched.TIE_SMALLER, kvsched.FEAS_PROFILE), *ctx.simulate(rows, s, o, M)]
    python.append(ctx.argmin(python[4]))
    for a, b in zip(native, python):
        assert a.dtype == b.dtype and a.device == b.device and a.shape == b.shape and torch.equal(a, b)
    ctx.close()


def test_what_is_refused():
    import torch
    from paper_2508_06133_amd import kvsched

    _, _, _, (s, o, rows) = _instance(40, 6)
    ctx = kvsched.Context(0)
    for bad in (s.long(), s.cpu(), torch.stack([s, s], 1)[:, 0]):
        for call in (lambda: ctx.sortedF(bad, o, 900), lambda: ctx.sortedF(s, bad, 900), lambda: ctx.simulate(rows, bad, o, 900),
                     lambda: ctx.simulate(rows, s, bad, 900), lambda: ctx.simulate(rows.t(), s, o, 900), lambda: ctx.argmin(s)):
            with pytest.raises(TypeError):
                call()
    with pytest.raises(ValueError):  # one row without its dimension
        ctx.simulate(rows[0], s, o, 900)
    for call in (lambda: ctx.sortedF(s, o, 1 << 30), lambda: ctx.simulate(rows, s, o, 1 << 30)):
        with pytest.raises(kvsched.KvschedError) as e:
            call()
        assert e.value.code == -2
    with pytest.raises(kvsched.KvschedError) as e:
        ctx.sortedF(s, o, 900, 7)
    assert e.value.code == -1
    ctx.close()
    with pytest.raises(kvsched.KvschedError) as e:  # after close()
        ctx.simulate(rows, s, o, 900)
    assert e.value.code == -1


def test_a_subclass_and_another_stream():
    import torch
    from paper_2508_06133_amd import kvsched

    class Lengths(torch.Tensor):
        pass

    s_h, o_h, rows_h, (s, o, rows) = _instance(120, 5)
    ctx = kvsched.Context(0)
    assert kvsched._host.sortedF(ctx._address, s.as_subclass(Lengths), o, 900, 0, 0, 0) is None  # (left to the Python path)
    order_o, _, _ = oracle.sortedF(s_h, o_h, 900)
    tel_o, _ = oracle.simulate_many(s_h, o_h, 900, rows_h)
    assert (torch.as_tensor(ctx.sortedF(s.as_subclass(Lengths), o, 900)[0]).cpu().numpy() == order_o).all()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        order, tel = ctx.sortedF(s, o, 900)[0], ctx.simulate(rows, s, o, 900)[0]
        best = ctx.argmin(tel)
    side.synchronize()
    assert (order.cpu().numpy() == order_o).all() and (tel.cpu().numpy() == tel_o).all() and best.tolist()[1] == int(tel_o.min())
    ctx.close()
