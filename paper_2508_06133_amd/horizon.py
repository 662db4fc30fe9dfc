"""Receding-horizon driver over libkvsched (offline form: every request present at round 0).

The loop only draws the window's moves and reads back six numbers per re-plan; the planning,
the move, the timeline and the commit point are computed by kvsched_horizon_step on the GPU.
"""
from __future__ import annotations

import numpy as np
import torch

from . import workloads


def receding_horizon(ctx, s, o, M, base_order, window: int = 512, complete_every: int = 256, moves_per_window: int = 65536,
                     rng: np.random.Generator | None = None, keep_tel: bool = False, max_steps: int | None = None,
                     keep_completion: bool = False):
    """-> (final order tensor, completion rounds tensor, list of per-step records).

    Each record: dict(lo, hi, best, best_tel, base_tel, committed, completed, T[, tel][, completion])."""
    rng = np.random.default_rng(0) if rng is None else rng
    n = int(base_order.shape[0])
    dev = base_order.device
    order = base_order.clone()
    completion = torch.empty(n, dtype=torch.int32, device=dev)
    committed, completed, log = 0, 0, []
    lazy = hasattr(ctx, "horizon_completion")  # (a stand-in for the context may offer the step alone)
    ahead = None  # (generator state before the draw, window length, moves relative to the window's start)
    while committed < n and (max_steps is None or len(log) < max_steps):
        lo, hi = committed, min(n, committed + window)
        if ahead is not None and ahead[1] == hi - lo:
            moves = ahead[2]
        else:
            if ahead is not None:  # the window came out shorter than expected: the draw has to be its own
                rng.bit_generator.state = ahead[0]
            moves = workloads.window_moves(rng, moves_per_window, 0, hi - lo)
        moves[:, 1:] += lo
        # The completion rounds of every request are wanted of the last order only (unless the caller keeps them all);
        # asking for them makes the step place the whole timeline.
        want = keep_completion or not lazy or (max_steps is not None and len(log) + 1 == max_steps)
        tel, res = ctx.horizon_step(order, torch.from_numpy(moves).to(dev), s, o, M, completed, complete_every,
                                    want_tel=keep_tel, completion_out=completion if want else None)
        # while the GPU works: the next window's moves (their positions relative to its start depend on its length
        # alone, which is nearly always this one's)
        ahead = (rng.bit_generator.state, hi - lo, workloads.window_moves(rng, moves_per_window, 0, hi - lo))
        r = [int(x) for x in res.cpu().numpy()]  # synchronises
        rec = dict(lo=lo, hi=hi, best=r[0], best_tel=r[1], base_tel=r[2], committed=r[3], completed=r[4], T=r[5])
        if keep_tel:
            rec["tel"] = tel.cpu().numpy()
        if keep_completion:  # completion rounds of the chosen order, by request id
            rec["completion"] = completion.cpu().numpy()
        log.append(rec)
        if r[0] < 0:
            rng.bit_generator.state = ahead[0]
            raise RuntimeError("receding_horizon: the order or the instance is malformed (see device_status)")
        committed, completed = r[3], r[4]
    if ahead is not None:  # (a draw that was not used is given back)
        rng.bit_generator.state = ahead[0]
    if log and not want:
        ctx.horizon_completion(order, o, completion)  # all positions committed: all of them are there
    return order, completion, log
