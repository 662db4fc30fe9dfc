"""The work that users of libkvsched have it do, as cases to be timed.

A case names one use of the library (its "kind"), the distribution the request lengths come from and
the sizes; every case goes through the public entry points of paper_2508_06133_amd.kvsched.Context (and
horizon.receding_horizon) as a scheduler program calls them.

  plan       Sorted-F order, the timelines of a set of candidate orders around it, the best of them
  neighbor   one local-search step: swap / insert moves anywhere in the order
  horizon    a whole receding-horizon run: re-plan, commit, re-plan
  sorted     the Sorted-F order under the simultaneous-start memory constraint
  swap       Phase 1 by Local Swap Search
  exact      Phase 1 by exact batches
  online     request streams under Poisson arrivals and three policies
  predicted  candidate orders under interval predictions of the decode lengths

The sizes of the listed cases are those of the five workload configurations and of bench.py.  Lengths are
drawn as in paper_2508_06133_amd.workloads, from a seed of the caller's.
"""
import functools
import itertools
import math

import numpy as np
import torch

from paper_2508_06133_amd import horizon, kvsched, workloads

DEVICE = "cuda:0"
MAX_DECODE = {"tiny": 8, "chat": 2048, "mixed": 2048, "bimodal": 4096}  # what the distributions are clipped to
LARGEST_REQUEST = {"tiny": 16, "chat": 4096, "mixed": 8692, "bimodal": 8192}  # prompt + decode
MAX_O = 14336  # scaled decode lengths are capped here
POLICIES = ((kvsched.PLANNER_ARRIVAL, 1, 0, 0, 0), (kvsched.PLANNER_SHORTEST_DECODE, 1, 0, 0, 0),
            (kvsched.PLANNER_SORTED_F, 10, 300, 1, 2))  # planner, period, window, growth trigger


def listed():
    return [
        # a scheduler orders a short backlog and asks when its requests will be done: the smallest calls
        dict(name="score_one", kind="plan", lengths="chat", n=61, M=16384, rows=1, swaps=1, scale=1, bound=False),
        # configuration 1: every order of eight requests beside the Sorted-F order
        dict(name="plan_exhaustive", kind="plan", lengths="tiny", n=8, M=48, rows=0, swaps=1, scale=1, bound=True),
        # configuration 2: short conversations, with the library finding the longest decode itself
        dict(name="plan_chat", kind="plan", lengths="chat", n=200, M=16384, rows=4096, swaps=1, scale=1, bound=False),
        # configuration 3, the headline workload: neighbours of the order and random restarts
        dict(name="plan_mixed", kind="plan", lengths="mixed", n=2000, M=131072, rows=16384, swaps=1, scale=1, bound=True),
        # configuration 5: a very long backlog of extreme requests, strongly perturbed orders
        dict(name="plan_bimodal", kind="plan", lengths="bimodal", n=100000, M=2097152, rows=1025, swaps=64, scale=1,
             bound=True),
        # a local-search step on configuration 3's backlog with answers four times as long
        dict(name="neighbor_long", kind="neighbor", lengths="mixed", n=2000, M=131072, moves=8191, scale=4, bound=False),
        # configuration 4's loop (windows of 512, a new plan every 256 completions) with a quarter of its moves
        dict(name="horizon_run", kind="horizon", lengths="mixed", n=10000, M=1048576, moves=16384, window=512, every=256),
        # Phase 1 on configuration 4's backlog under the constraint of Algorithm 1
        dict(name="sorted_profile", kind="sorted", lengths="mixed", n=10000, M=1048576, profile=True, larger=True),
        # Phase 1 by Local Swap Search on configuration 3's backlog
        dict(name="local_swap", kind="swap", lengths="mixed", n=2000, M=131072, alpha_num=0, alpha_den=1),
        # Phase 1 by exact batches on configuration 2's backlog
        dict(name="exact_dp", kind="exact", lengths="chat", n=200, M=16384, profile=False),
        # the Poisson experiment: ten loads, twenty arrival sequences each, three policies
        dict(name="online_grid", kind="online", sequences=20, rounds=4000),
        # configuration 3's candidates when only intervals of the decode lengths are known
        dict(name="predicted", kind="predicted", lengths="mixed", n=2000, M=131072, rows=4096, gamma=0.6, per_row=False,
             bound=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _budget(rng, lengths, n):
    """A KV budget of a few tens of tokens per waiting request, as in the configurations, but one that
    holds the largest request at least once and a half."""
    per_request = {"tiny": (3, 8), "chat": (30, 120), "mixed": (40, 120), "bimodal": (20, 60)}[lengths]
    return max(int(1.5 * LARGEST_REQUEST[lengths]), int(n * rng.uniform(*per_request)))


def draw(rng):
    kind = rng.choice(["plan", "plan", "neighbor", "horizon", "sorted", "swap", "exact", "online", "predicted"])
    if kind == "plan":
        lengths = rng.choice(["chat", "mixed", "bimodal"])
        n = _log_int(rng, 24, 100000 if lengths == "bimodal" else 12000)
        rows = max(1, min(_log_int(rng, 1, 32768), (100_000_000 if lengths == "bimodal" else 32_000_000) // n))
        return dict(kind=kind, lengths=lengths, n=n, M=_budget(rng, lengths, n), rows=rows, swaps=rng.choice([1, 1, 8, 64]),
                    scale=rng.choice([1, 1, 2, 4]) if lengths != "bimodal" else 1, bound=rng.random() < 0.5)
    if kind == "neighbor":
        lengths = rng.choice(["chat", "mixed"])
        n = _log_int(rng, 100, 8000)
        return dict(kind=kind, lengths=lengths, n=n, M=_budget(rng, lengths, n),
                    moves=min(_log_int(rng, 256, 32768), 33_000_000 // n), scale=rng.choice([1, 1, 2, 4]),
                    bound=rng.random() < 0.5)
    if kind == "horizon":
        n = _log_int(rng, 500, 10000)
        return dict(kind=kind, lengths="mixed", n=n, M=_budget(rng, "mixed", n), moves=_log_int(rng, 512, 16384),
                    window=rng.choice([128, 256, 512]), every=256)
    if kind == "sorted":
        lengths = rng.choice(["chat", "mixed", "bimodal"])
        n = _log_int(rng, 64, 40000)
        return dict(kind=kind, lengths=lengths, n=n, M=_budget(rng, lengths, n), profile=rng.random() < 0.6,
                    larger=rng.random() < 0.7)
    if kind == "swap":
        lengths = rng.choice(["chat", "mixed"])
        n = _log_int(rng, 64, 10000)
        num, den = rng.choice([(0, 1), (0, 1), (13, 1000), (1, 1), (5, 1)])
        return dict(kind=kind, lengths=lengths, n=n, M=_budget(rng, lengths, n), alpha_num=num, alpha_den=den)
    if kind == "exact":
        if rng.random() < 0.3:
            return dict(kind=kind, lengths="tiny", n=_log_int(rng, 20, 200), M=rng.randint(48, 200),
                        profile=rng.random() < 0.3)
        return dict(kind=kind, lengths="chat", n=_log_int(rng, 30, 220), M=_log_int(rng, 6144, 16384),
                    profile=rng.random() < 0.3)
    if kind == "online":
        return dict(kind=kind, sequences=_log_int(rng, 1, 20), rounds=_log_int(rng, 500, 4000))
    n = _log_int(rng, 100, 2400)
    lengths = rng.choice(["chat", "mixed"])
    return dict(kind=kind, lengths=lengths, n=n, M=_budget(rng, lengths, n), rows=_log_int(rng, 16, 4096),
                gamma=round(rng.uniform(0.3, 0.95), 3), per_row=rng.random() < 0.25, bound=rng.random() < 0.5)


# ------------------------------------------------------------------------------------------- inputs


@functools.lru_cache(maxsize=None)
def _context(bound):
    """One context per bound on the decode lengths (0: the library looks for the longest itself), kept for
    the whole program, as a scheduler keeps it from one backlog to the next."""
    ctx = kvsched.Context(0)
    ctx.set_o_max(bound)
    return ctx


def _lengths(rng, kind, n, scale=1):
    if kind == "tiny":
        return rng.integers(1, 9, n).astype(np.int32), rng.integers(1, 9, n).astype(np.int32)
    if kind == "bimodal":
        s = np.where(rng.random(n) < 0.5, 1, 4096)
        o = np.where(rng.random(n) < 0.5, 4096, 1)
    else:
        s = np.clip(np.rint(rng.lognormal(np.log(128.0), 0.8, n)), 4, 2048)
        o = np.clip(np.rint(rng.lognormal(np.log(200.0), 0.9, n)), 1, 2048)
        if kind == "mixed":
            is_long = rng.random(n) < 0.3
            s = np.where(is_long, rng.integers(2048, 8193, n), s)
            o = np.where(is_long, rng.integers(100, 501, n), o)
    return s.astype(np.int32), np.minimum(o * scale, MAX_O).astype(np.int32)


def _candidates(base, rows, swaps, seed):
    """Row 0 is the base order; the others exchange `swaps` random pairs of positions of it in turn, and one
    in 64 is a random permutation (a restart) when single exchanges are drawn."""
    n = base.shape[0]
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    orders = base.repeat(rows, 1)
    at = torch.arange(1, rows, device=DEVICE)
    for _ in range(swaps if rows > 1 else 0):
        ij = torch.randint(0, n, (2, rows - 1), generator=gen, device=DEVICE)
        a, b = orders[at, ij[0]], orders[at, ij[1]]
        orders[at, ij[0]], orders[at, ij[1]] = b, a
    restarts = rows // 64 if swaps == 1 else 0
    if restarts:
        keys = torch.rand((restarts, n), generator=gen, device=DEVICE)
        orders[rows - restarts:] = torch.argsort(keys, dim=1).to(torch.int32)
    return orders


def _plan_state(case, st, seed):
    s, o, M = st["s"], st["o"], st["M"]
    order = st["ctx"].sortedF(s, o, M)[0]
    if case["rows"]:
        st["orders"] = _candidates(order, case["rows"], case["swaps"], seed)
    else:
        every = torch.tensor(list(itertools.permutations(range(case["n"]))), dtype=torch.int32, device=DEVICE)
        st["orders"] = torch.cat([every, order[None, :]])


def _expected_requests(case):
    return workloads.online_lambda_star() * case["rounds"] * case["sequences"] * sum(workloads.ONLINE_RHO)


def prepare(case, seed):
    kind = case["kind"]
    rng = np.random.default_rng(seed)
    st = {"case": case, "seed": seed}
    if kind == "online":
        a_all, s_all, o_all, desc = [], [], [], []
        first = out = 0
        for k, rho in enumerate(workloads.ONLINE_RHO):
            for q in range(case["sequences"]):
                a, s, o, M = workloads.online_instance(seed * 1000 + 50 * k + q, rho, T=case["rounds"])
                a_all.append(a), s_all.append(s), o_all.append(o)
                for policy in POLICIES:
                    desc.append([first, len(a), *policy, out])
                    out += len(a)
                first += len(a)
        st.update(ctx=_context(MAX_DECODE["mixed"]), M=M, cap=512, desc=torch.tensor(desc, dtype=torch.int32, device=DEVICE))
        for name, v in (("a", a_all), ("s", s_all), ("o", o_all)):
            st[name] = torch.from_numpy(np.concatenate(v)).to(DEVICE)
        # an output buffer kept from one batch of streams to the next: room for more requests than expected
        room = int(1.25 * len(POLICIES) * _expected_requests(case)) + 4096
        assert out <= room
        st["completion"] = torch.zeros(room, dtype=torch.int32, device=DEVICE)
        return st
    n, scale = case["n"], case.get("scale", 1)
    s, o = _lengths(rng, case["lengths"], n, scale)
    bound = min(MAX_DECODE[case["lengths"]] * scale, MAX_O) if case.get("bound") else 0
    st.update(ctx=_context(bound), M=case["M"] * scale, s=torch.from_numpy(s).to(DEVICE), o=torch.from_numpy(o).to(DEVICE))
    if kind == "plan":
        _plan_state(case, st, seed)
    elif kind == "neighbor":
        st["order"] = st["ctx"].sortedF(st["s"], st["o"], st["M"])[0]
        st["moves"] = torch.from_numpy(workloads.moves_anywhere(rng, case["moves"], n)).to(DEVICE)
    elif kind == "horizon":
        st["order"] = st["ctx"].sortedF(st["s"], st["o"], st["M"])[0]
    elif kind == "predicted":
        # (the estimates start at or below the true lengths: the bound covers both)
        lower, _ = workloads.prediction_intervals(seed, s, o, st["M"], case["gamma"])
        est = torch.from_numpy(lower).to(DEVICE)
        order = st["ctx"].sortedF(st["s"], est, st["M"])[0]
        st["orders"] = _candidates(order, case["rows"], 1, seed)
        if case["per_row"]:  # every row its own prediction between the lower bound and the truth
            gen = torch.Generator(device=DEVICE).manual_seed(seed + 1)
            u = torch.rand((case["rows"], n), generator=gen, device=DEVICE)
            est = (est + (u * (st["o"] - est + 1)).to(torch.int32)).clamp(max=st["o"]).to(torch.int32).contiguous()
        st["est"] = est
    return st


# -------------------------------------------------------------------------------------- one pass


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "online":
        return ctx.online(st["desc"], st["a"], st["s"], st["o"], st["M"], st["completion"], backlog_cap=st["cap"])
    s, o, M = st["s"], st["o"], st["M"]
    if kind == "plan":
        order, ends, F, nb = ctx.sortedF(s, o, M)
        tel, completion = ctx.simulate(st["orders"], s, o, M)
        best = ctx.argmin(tel) if case["rows"] != 1 else tel
        return order, ends, F, nb, tel, completion, best
    if kind == "neighbor":
        return ctx.best_neighbor(st["order"], st["moves"], s, o, M)
    if kind == "horizon":
        order, completion, log = horizon.receding_horizon(
            ctx, s, o, M, st["order"], window=case["window"], complete_every=case["every"],
            moves_per_window=case["moves"], rng=np.random.default_rng(st["seed"]))
        steps = np.zeros((case["n"] // case["every"] + 2, 8), dtype=np.int64)  # (as many re-plans as there can be)
        steps[:len(log)] = [[r[k] for k in sorted(r)] for r in log]
        return order, completion, steps
    if kind == "sorted":
        return ctx.sortedF(s, o, M, kvsched.TIE_LARGER if case["larger"] else kvsched.TIE_SMALLER,
                           kvsched.FEAS_PROFILE if case["profile"] else kvsched.FEAS_SUM_OF_PEAKS)
    if kind == "swap":
        if case["alpha_num"] == 0:
            return ctx.local_swap(s, o, M)
        return ctx.phase1_G(kvsched.SOLVER_LOCAL_SWAP, s, o, M, (case["alpha_num"], case["alpha_den"]))
    if kind == "exact":
        return ctx.exact_dp(s, o, M, kvsched.FEAS_PROFILE if case["profile"] else kvsched.FEAS_SUM_OF_PEAKS)
    return ctx.simulate_predicted(st["orders"], s, o, st["est"], M)


def work(case):
    """Bytes: every input and output once.  Operations: one test and one commitment per request and timeline
    (exact batches: one comparison per request, batch size and load)."""
    kind = case["kind"]
    if kind == "online":
        requests = _expected_requests(case)
        return {"bytes": requests * (12 + 3 * 4), "flops": 2 * 3 * requests}
    n = case["n"]
    phase1 = 8 * n + 16 * n + 4  # lengths in; order, batch ends and metric out
    if kind == "plan":
        rows = case["rows"] or math.factorial(n) + 1
        return {"bytes": phase1 + 8 * n + rows * (8 * n + 8), "flops": 2 * rows * n + n}
    if kind == "neighbor":
        return {"bytes": 12 * n + case["moves"] * (12 + 8), "flops": 2 * case["moves"] * n}
    if kind == "horizon":
        replans = max(1, n // case["every"])
        return {"bytes": 16 * n + replans * case["moves"] * 12, "flops": 2 * replans * case["moves"] * n / 2}
    if kind in ("sorted", "swap"):
        return {"bytes": phase1, "flops": n * max(1.0, math.log2(n))}
    if kind == "exact":
        batch = max(1, min(n, case["M"] // (9 if case["lengths"] == "tiny" else 300)))
        return {"bytes": phase1, "flops": float(n) * batch * case["M"]}
    rows = case["rows"]
    return {"bytes": 8 * n + 4 * n * (rows if case["per_row"] else 1) + rows * (8 * n + 12), "flops": 2 * rows * n}


def tolerance(case):
    """Everything is integers except the metric of a batch, one fp64 division."""
    if case["kind"] in ("plan", "sorted", "swap", "exact"):
        return {"rel": 1e-12, "max": 1e-12}
    return "exact"
