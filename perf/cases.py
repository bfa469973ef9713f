"""The measured work of libfleetsieve: what a fleet planner has it do, through
the Python binding's public calls, on inputs already resident on the GPU.

Every case names one kind of call and its sizes:

* ``round``      one planning step of one fleet: the certificate, then the
                 acquisition score (``certify`` + ``ScorePlan``);
* ``score``      the acquisition score of many reveal orders (``ScorePlan``);
                 ``floors`` adds critical classes with served-rate floors;
* ``solve``      dense allocation solves of point realisations
                 (``solve_batch``), ``solve_lex`` the same under the whole
                 lexicographic objective (``solve_batch_lex``);
* ``score_lex``  the stage-wise score (``ScoreLexPlan``);
* ``loop``       Algorithm 1 for many trajectories (``profile_loop``), with
                 or without the interval refit;
* ``policy``     the class-policy step: both reductions, then the score.

Inputs follow the recipes of ``paper_2608_19659_amd.synth`` (capacity knee at
TP4, tails growing with the load, capacities on a 1/64 req/s grid, a random
number of revealed cells per order, samples uniform inside the intervals),
drawn from the seed here so that every seed is another problem; demands are
scaled until the budget binds, as a fleet's does that needs planning.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_19659_amd import fleetsieve as fs
from paper_2608_19659_amd.synth import SLO_CHOICES, TAIL_TP_FACTOR, Problem, q64

TP_SETS = {3: [2, 4, 8], 4: [1, 2, 4, 8], 5: [1, 2, 4, 8, 16]}
EPS = 0.05


def listed():
    return [
        # One fleet of two classes on 16 GPUs between two measurements: the
        # smallest calls, all latency and launches.
        dict(name="round-2class-G16", kind="round", K=2, nt=4, G=16, B=3, dlo=2.0, dhi=4.0, O=1, E=8, S=64),
        # 200 random reveal orders of the two-class, 16-GPU fleet.
        dict(name="score-2class-G16", kind="score", K=2, nt=4, G=16, B=6, dlo=3.0, dhi=4.0, O=200, E=0, S=1024),
        # The benchmark's workload: four classes on 64 GPUs.
        dict(name="score-4class-G64", kind="score", K=4, nt=4, G=64, B=8, dlo=1.0, dhi=20.0, O=16, E=0, S=4096),
        # The largest sampled workload: eight classes on 256 GPUs, 67 M samples.
        dict(name="score-8class-G256", kind="score", K=8, nt=4, G=256, B=8, dlo=0.5, dhi=50.0, O=64, E=0, S=4096),
        # A large fleet: 16 classes on 1024 GPUs, where the tables are the work.
        dict(name="score-16class-G1024", kind="score", K=16, nt=5, G=1024, B=12, dlo=1.0, dhi=200.0, O=4, E=0, S=256),
        # Critical classes with served-rate floors, at sizes that are no
        # multiple of anything.
        dict(name="score-floors-5class-G48", kind="score", K=5, nt=4, G=48, B=7, dlo=0.6, dhi=12.0, O=12, E=0, S=999,
             floors=True),
        # What-if solves of sampled tables of the four-class fleet.
        dict(name="solve-4class-G64", kind="solve", K=4, nt=4, G=64, B=8, dlo=1.0, dhi=20.0, O=16, n=65536),
        # The same under the whole objective (goodput, then fewest GPUs).
        dict(name="solve-lex-4class-G64", kind="solve_lex", K=4, nt=4, G=64, B=8, dlo=1.0, dhi=20.0, O=16, n=65536),
        # The stage-wise score, with the 64 samples a planner takes per cell.
        dict(name="score-lex-4class-G64", kind="score_lex", K=4, nt=4, G=64, B=8, dlo=1.0, dhi=20.0, O=16, E=0, S=64),
        # Algorithm 1 over 200 reveal orders until every one is certified.
        dict(name="loop-2class-G16", kind="loop", K=2, nt=4, G=16, B=6, dlo=3.0, dhi=4.0, O=200, E=0, S=1024,
             refit=False),
        # Algorithm 1 with its fit step on tables that satisfy the prior.
        dict(name="loop-refit-4class-G64", kind="loop", K=4, nt=4, G=64, B=8, dlo=1.0, dhi=20.0, O=16, E=0, S=4096,
             refit=True),
        # The class-policy step: two tail metrics and a success floor.
        dict(name="policy-4class-G64", kind="policy", K=4, nt=4, G=64, B=8, dlo=1.0, dhi=20.0, O=16, E=0, S=4096),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: the same kinds of call over 2 to 16 classes, 16 to 1024
    GPUs (less where a whole-objective solve is quadratic in them), 3 to 12
    load levels, 1 to 200 orders, 1 to 4096 samples, cut to the listed cases'
    work."""
    kind = rng.choice(["round", "score", "score", "floors", "solve", "solve_lex", "score_lex", "loop", "policy"])
    big = kind in ("score", "floors", "solve", "policy")
    K = rng.randint(2, 16 if big else 6)
    G = _log(rng, 16, 1024 if big else 512 if kind == "solve_lex" else 96)
    K = min(K, G // 6)
    nt, B = rng.choice([3, 4, 4, 5]), rng.randint(3, 12 if big else 8)
    c = dict(kind="score" if kind == "floors" else kind, K=K, nt=nt, G=G, B=B, dlo=round(0.06 * G / K, 3),
             dhi=round(1.25 * G / K, 3), O=_log(rng, 1, 200))
    N = K * nt * B
    if kind in ("solve", "solve_lex"):
        c["O"] = 1 + c["O"] % 16
        most = 65536 * 4 * 64 // (K * G) if kind == "solve" else 65536 * 4 * 64 * 64 // (K * G * G)
        c["n"] = _log(rng, 1, max(1, min(65536, most)))
        return c
    c["E"] = 0 if rng.random() < 0.7 else rng.randint(1, N)
    E = c["E"] or N
    if kind == "round":
        c["O"] = rng.randint(1, 4)
        c["S"] = _log(rng, 1, 512)
        return c
    c["S"] = _log(rng, 16, 4096)
    per = {"score": 64 << 20, "policy": 8 << 20, "floors": 4e8 / (K * G), "score_lex": 16 * 128 * 64,
           "loop": 2e8 / E}[kind]
    c["O"] = max(1, min(c["O"], int(per // (16 * E))))
    c["S"] = max(1, min(c["S"], int(per // (c["O"] * E))))
    if kind == "score_lex":  # interval tables: 2 O K intervals of K-1 layers of G costs
        c["O"] = max(1, min(c["O"], int(16 * 4 ** 3 * 64 ** 3 / (K ** 3 * G ** 3))))
    if kind == "floors":
        c["floors"] = True
    if kind == "loop":
        c["refit"] = rng.random() < 0.5
    return c


# ------------------------------------------------------------------ inputs --
def _geometry(c):
    tp = np.array(TP_SETS[c["nt"]])
    levels = 2.0 ** (np.arange(c["B"]) - math.ceil(c["B"] / 3))
    return c["K"], tp, c["B"], levels


def _knee(rng, shape, tp, lo, hi):
    """Capacities [*shape, T] on the grid, per GPU strictly largest at TP4."""
    k4 = tp.tolist().index(4)
    out, todo = np.zeros((*shape, len(tp))), np.ones(shape, bool)
    while todo.any():
        caps = q64(rng.uniform(lo, hi, size=(int(todo.sum()), len(tp))))
        per = caps / tp
        ok = np.all(np.delete(per, k4, axis=1) < per[:, k4:k4 + 1], axis=1)
        idx = np.argwhere(todo)[ok]
        out[tuple(idx.T)] = caps[ok]
        todo[tuple(idx.T)] = False
    return out


def _unimodal(rng, shape, tp, lo, hi):
    """Capacities [*shape, T] on the grid, per GPU rising to TP4, then falling."""
    k4 = tp.tolist().index(4)
    out, todo = np.zeros((*shape, len(tp))), np.ones(shape, bool)
    while todo.any():
        n = int(todo.sum())
        g = np.zeros((n, len(tp)))
        g[:, k4] = rng.uniform(lo, hi, n) / 4.0
        for t in range(k4 - 1, -1, -1):
            g[:, t] = g[:, t + 1] * rng.uniform(0.55, 0.95, n)
        for t in range(k4 + 1, len(tp)):
            g[:, t] = g[:, t - 1] * rng.uniform(0.55, 0.95, n)
        caps = q64(g * tp)
        per = caps / tp
        ok = np.all(np.diff(per[:, :k4 + 1]) >= 0, axis=1) & np.all(np.diff(per[:, k4:]) <= 0, axis=1)
        idx = np.argwhere(todo)[ok]
        out[tuple(idx.T)] = caps[ok]
        todo[tuple(idx.T)] = False
    return out


def _host_tau(p, cap, tail):
    """The max-min optimum of one table: merging nondecreasing tables, entry g
    of the result is the entry of rank g in their sorted union."""
    r = np.arange(1, p.budget + 1)
    cap, tail = (a.reshape(p.n_classes, p.n_tp, p.n_levels) for a in (cap, tail))
    joint = None
    for i in range(p.n_classes):
        table = np.zeros(p.budget + 1)
        b = np.searchsorted(p.levels, p.demand[i] / r)
        for t, g in enumerate(p.tp):
            n = p.budget // int(g)
            fits = b[:n] < p.n_levels
            at = np.minimum(b[:n], p.n_levels - 1)
            f = np.where(fits & (tail[i, t, at] <= p.slo[i]), np.minimum(1.0, r[:n] * cap[i, t, at] / p.demand[i]), 0.0)
            np.maximum.at(table, int(g) * r[:n], f)
        table = np.maximum.accumulate(table)
        joint = table if joint is None else np.sort(np.concatenate([joint, table]))[: p.budget + 1]
    return joint[-1]


def _host(c, seed, again=0):
    """The problem, the orders' intervals and the hidden truth (host arrays)."""
    K, tp, B, levels = _geometry(c)
    T, O, N = len(tp), c["O"], K * len(tp) * B
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence([seed, K, c["G"], N, again])))
    demand = rng.uniform(c["dlo"], c["dhi"], K).astype(np.float32)
    slo = np.full(K, 30.0, np.float32) if K == 2 else rng.choice(np.array(SLO_CHOICES, np.float32), K)
    problem = Problem(tp=tp, levels=levels, demand=demand, slo=slo, budget=c["G"])
    small = K == 2
    lo, hi = (0.2, 3.0) if small else (0.1, 5.0)
    wide = (0.02, 0.5) if K >= 8 else (0.05, 0.3)
    tail_w = (0.02, 0.5) if K >= 8 else (0.1, 0.4)
    rho = np.array([TAIL_TP_FACTOR[int(t)] for t in tp])
    median = (slo.astype(np.float64) / 3.0)[:, None, None] * (1.0 + levels) ** (1.5 if small else 1.0) * rho[:, None]
    tail = (median * np.exp((0.4 if small else 0.5) * rng.standard_normal((K, T, B)))).astype(np.float32)
    if c.get("refit"):  # the truth first, then intervals around it
        tcap = np.moveaxis(_unimodal(rng, (K, B), tp, lo, hi), 2, 1).reshape(N)
        ttail = np.maximum.accumulate(tail, axis=2).reshape(N)
        cl = np.minimum(q64(tcap * (1.0 - rng.uniform(*wide, N))), tcap)
        ch = np.maximum(q64(tcap * (1.0 + rng.uniform(*wide, N))), tcap)
        tl = np.minimum((ttail / (1.0 + rng.uniform(*tail_w, N))).astype(np.float32), ttail)
        th = np.maximum((ttail * (1.0 + rng.uniform(*tail_w, N))).astype(np.float32), ttail)
    else:
        cl = np.moveaxis(_knee(rng, (K, B), tp, lo, hi), 2, 1).reshape(N)
        ch = np.maximum(q64(cl * (1.0 + rng.uniform(*wide, N))), cl)
        tl = tail.reshape(N)
        th = np.maximum((tl * (1.0 + rng.uniform(*tail_w, N))).astype(np.float32), tl)
        tcap = cl + np.floor(rng.random(N) * (np.rint((ch - cl) * 64.0) + 1.0)) / 64.0
        ttail = np.clip(tl + rng.random(N).astype(np.float32) * (th - tl), tl, th)
    # the budget binds: demand up while every class is served in full, down
    # while one can't be served at all
    step, last = 1.5, 0
    for _ in range(20):
        tau = _host_tau(problem, cl, th)
        turn = 1 if tau >= 1.0 else -1 if tau <= 0.0 else 0
        if turn == 0:
            break
        step = step if turn != -last else math.sqrt(step)
        last, problem.demand = turn, (problem.demand * step ** turn).astype(np.float32)
    if turn < 0 and again < 8:  # a class that no cell serves at any load: another draw
        return _host(c, seed, again + 1)
    if c.get("floors"):  # every other class critical, at 5 to 50% of its demand
        share = np.where(np.arange(K) % 2 == 0, rng.uniform(0.05, 0.5, K), 0.0)
        problem.floor_rps = (problem.demand * share).astype(np.float32)
    # revealed cells: a random number of them per order, at the truth
    ms = np.argsort(rng.random((O, N)), axis=1).argsort(axis=1) < rng.integers(0, N, (O, 1))
    pick = lambda point, a: np.where(ms, point, a).astype(np.float32)  # noqa: E731
    iv = (pick(tcap, cl), pick(tcap, ch), pick(ttail, tl), pick(ttail, th), ms.astype(np.uint8))
    E = c.get("E") or N
    cand = np.sort(rng.permutation(N)[:E]).astype(np.int32)
    return problem, iv, cand, tcap.astype(np.float32), ttail.astype(np.float32), rng


def _inside(gen, lo, hi, shape, grid):
    """Uniform inside [lo, hi]: on the 1/64 req/s grid, or in binary32."""
    u = torch.rand(shape, generator=gen, device="cuda")
    if grid:
        k = torch.floor(u * (torch.round((hi - lo) * 64.0) + 1.0))
        return torch.minimum(lo + k / 64.0, hi)
    return torch.minimum(lo + u * (hi - lo), hi)


def _inputs(c, seed):
    """Everything a call reads, on the GPU (torch tensors), from the seed."""
    problem, iv, cand, tcap, ttail, rng = _host(c, seed)
    gen = torch.Generator("cuda").manual_seed(int(seed))
    d = dict(problem=problem, iv=fs.DeviceIntervals(*(torch.from_numpy(a).cuda() for a in iv)),
             cand=torch.from_numpy(cand).cuda())
    v, O = d["iv"], c["O"]
    if c["kind"] in ("solve", "solve_lex"):  # realisation j: every cell inside the intervals of order j mod O
        rows = torch.arange(c["n"], device="cuda") % O
        shape = (c["n"], problem.n_cells)
        d["cap"] = _inside(gen, v.cap_lo[rows], v.cap_hi[rows], shape, True)
        d["tail"] = _inside(gen, v.tail_lo[rows], v.tail_hi[rows], shape, False)
        return d
    at = d["cand"].long()
    shape = (O, len(cand), c["S"])
    side = lambda a: a[:, at][:, :, None]  # noqa: E731
    d["cap_s"] = _inside(gen, side(v.cap_lo), side(v.cap_hi), shape, True)
    d["tail_s"] = _inside(gen, side(v.tail_lo), side(v.tail_hi), shape, False)
    if c["kind"] == "loop":
        d["truth_cap"] = torch.from_numpy(np.tile(tcap, (O, 1))).cuda()
        d["truth_tail"] = torch.from_numpy(np.tile(ttail, (O, 1))).cuda()
    if c["kind"] == "policy":
        K, tp, B, levels = _geometry(c)
        N = problem.n_cells
        limit = np.stack([problem.slo, problem.slo / 10.0], axis=1).astype(np.float32)
        rho = np.array([TAIL_TP_FACTOR[int(t)] for t in tp])
        med = (limit[:, 1] / 4.0)[:, None, None] * (1.0 + levels) ** 0.5 * rho[:, None]
        tl = (med * np.exp(0.4 * rng.standard_normal((K, len(tp), B)))).astype(np.float32).reshape(N)
        th = (tl * (1.0 + rng.uniform(0.1, 0.4, N))).astype(np.float32)
        sh = (1.0 - 10.0 ** -rng.uniform(2.0, 4.0, N)).astype(np.float32)
        sl = np.maximum(0.0, sh - rng.uniform(0.0, 0.005, N)).astype(np.float32)
        tl, th, sl, sh = (torch.from_numpy(a).cuda().expand(O, N) for a in (tl, th, sl, sh))
        ms = v.measured.bool()
        th, sl = torch.where(ms, tl, th), torch.where(ms, sh, sl)
        # rows 0..O-1 the conservative side, O..2O-1 the optimistic one
        d["tails"] = torch.stack([torch.cat([v.tail_hi, v.tail_lo]), torch.cat([th, tl])], dim=-1).contiguous()
        d["succ"] = torch.cat([sl, sh]).contiguous()
        ttft_s = _inside(gen, side(tl), side(th), shape, False)
        d["metric_s"] = torch.stack([d["tail_s"], ttft_s], dim=-1).contiguous()
        d["succ_s"] = _inside(gen, side(sl), side(sh), shape, False)
        d["limit"], d["success_min"] = limit, np.full(K, 0.99, np.float32)
    return d


class _Policy:
    def __init__(self, limit, success_min):
        self.limit, self.success_min = limit, success_min


def prepare(case, seed):
    d = _inputs(case, seed)
    ctx = fs.Context(0)
    s = dict(d, kind=case["kind"], ctx=ctx, refit=case.get("refit", False))
    kind, p = case["kind"], d["problem"]
    if kind in ("round", "score"):
        s["plan"] = fs.ScorePlan(ctx, p, d["iv"], d["cand"], d["cap_s"], d["tail_s"])
    elif kind == "score_lex":
        s["plan"] = fs.ScoreLexPlan(ctx, p, d["iv"], d["cand"], d["cap_s"], d["tail_s"])
    elif kind == "policy":  # a problem whose limits are the pseudo-tails'
        pol = _Policy(d["limit"], d["success_min"])
        s["cells"] = fs.ReducePlan.cells(ctx, p, pol, d["tails"], d["succ"])
        s["samples"] = fs.ReducePlan.samples(ctx, p, pol, d["cand"], d["metric_s"], d["succ_s"])
        p0 = Problem(p.tp, p.levels, p.demand, np.zeros(p.n_classes, np.float32), p.budget)
        red, O, v = s["cells"].out, case["O"], d["iv"]
        iv = fs.DeviceIntervals(v.cap_lo, v.cap_hi, red[O:], red[:O], v.measured)
        s["plan"] = fs.ScorePlan(ctx, p0, iv, d["cand"], d["cap_s"], s["samples"].out)
    return s


def _scored(o):
    return dict(score=o.score, gap_now=o.gap_now, best=o.best)


def run(state):
    s, kind = state, state["kind"]
    ctx, p = s["ctx"], s["problem"]
    if kind == "score":
        return _scored(s["plan"].run())
    if kind == "round":
        c = fs.certify(ctx, p, s["iv"], EPS)
        return dict(_scored(s["plan"].run()), state=c.state, gap=c.gap, cons=c.cons, opt=c.opt)
    if kind == "solve":
        return fs.solve_batch(ctx, p, s["cap"], s["tail"])
    if kind == "solve_lex":
        return fs.solve_batch_lex(ctx, p, s["cap"], s["tail"])
    if kind == "score_lex":
        o = s["plan"].run()
        return dict(score_maxmin=o.score_maxmin, score_goodput=o.score_goodput, gap_maxmin=o.gap_maxmin,
                    gap_goodput=o.gap_goodput, best=o.best)
    if kind == "policy":
        cells, samples = s["cells"].run(), s["samples"].run()
        return dict(_scored(s["plan"].run()), cells=cells, samples=samples)
    o = fs.profile_loop(ctx, p, s["iv"], s["truth_cap"], s["truth_tail"], s["cand"], s["cap_s"], s["tail_s"], EPS,
                        refit=s["refit"])
    return dict(state=o.state, finished=o.finished, rounds=o.rounds, gpu_seconds=o.gpu_seconds, reveals=o.reveals,
                final=o.final, tau_truth=o.tau_truth, tau_oracle=o.tau_oracle)


# ------------------------------------------------------------ work, bounds --
def work(case):
    """Bytes: every input once (the samples of unmeasured candidates only,
    half of them on average, since measured ones are not solved) and every
    output once.  Operations: per sampled scenario about 20 (its options'
    ratios against the tables of the other classes), per dense solve the
    options' ratios and one pass over each class's table; a loop makes about
    one such round per eighth of its candidates."""
    c, kind = case, case["kind"]
    K, tp, B, _ = _geometry(c)
    N, O = K * len(tp) * B, c["O"]
    P = sum(c["G"] // int(t) for t in tp)
    solve = 4 * K * P + 8 * K * c["G"]
    if kind in ("solve", "solve_lex"):
        return dict(bytes=c["n"] * (8 * N + 3 * K + 9 + (8 if kind == "solve_lex" else 0)),
                    flops=c["n"] * (solve + (2 * K * P if kind == "solve_lex" else 0)))
    E = c.get("E") or N
    half = O * E * c["S"] // 2
    tables = O * N * 17 + 4 * E + O * E * 8 + O * 12
    flops = 20 * half + 2 * O * K * solve
    if kind == "policy":
        return dict(bytes=tables + O * N * 2 * 16 + 16 * O * E * c["S"] + 8 * half, flops=flops + 4 * O * E * c["S"])
    if kind == "score_lex":
        return dict(bytes=tables + 8 * half + 8 * O * E, flops=2 * flops)
    if kind == "loop":
        rounds = max(1, E // 8)
        return dict(bytes=tables + 8 * half + 8 * O * N + O * (3 * K + 30), flops=rounds * (flops // 2 + 4 * O * solve))
    extra = 2 * O * (3 * K + 9) + 12 * O if kind == "round" else 0
    return dict(bytes=tables + 8 * half + extra, flops=flops + (2 * O * solve if kind == "round" else 0))


def tolerance(case):
    """Every ratio is one multiply and one correctly rounded divide in
    binary32, every sum binary64 in a fixed order: the C ABI states the bits."""
    return "exact"


# ---------------------------------------------- the same results in 64 bits --
def _options(p):
    """(class, TP index, replicas, cost, level) of every option that exists."""
    rows = []
    for i in range(p.n_classes):
        for t, g in enumerate(p.tp):
            for r in range(1, p.budget // int(g) + 1):
                b = int(np.searchsorted(p.levels, np.float32(p.demand[i]) / np.float32(r)))
                if b < p.n_levels:
                    rows.append((i, t, r, int(g) * r, p.cell(i, t, b)))
    return np.array(rows, np.int64).reshape(-1, 5)


def _ratios(p, opt, cap, tail):
    """Ratio and served rate [n][options], 0 where the tail breaks the SLO."""
    at = torch.from_numpy(opt[:, 4]).cuda()
    lam = torch.from_numpy(p.demand[opt[:, 0]].astype(np.float64)).cuda()
    slo = torch.from_numpy(p.slo[opt[:, 0]].astype(np.float64)).cuda()
    rate = torch.minimum(cap.double()[:, at] * torch.from_numpy(opt[:, 2]).cuda(), lam)
    rate = torch.where(tail.double()[:, at] <= slo, rate, 0.0)
    return rate / lam, rate


def _class_tables(p, opt, ratio):
    """Best ratio of each class with at most g GPUs: [K][n][G + 1]."""
    tab = torch.zeros((p.n_classes, ratio.shape[0], p.budget + 1), dtype=torch.float64, device="cuda")
    for i in range(p.n_classes):
        cols = np.flatnonzero(opt[:, 0] == i)
        if len(cols):
            idx = torch.from_numpy(opt[cols, 3]).cuda().expand(ratio.shape[0], -1)
            tab[i].scatter_reduce_(1, idx, ratio[:, torch.from_numpy(cols).cuda()], "amax")
        tab[i] = torch.cummax(tab[i], dim=1).values
    return tab


def _maxmin(a, b):
    """The (max, min) convolution of nondecreasing tables [n][G + 1]: its
    entry g is the entry of rank g in their sorted union."""
    out = torch.cat([a, b], dim=1).sort(dim=1).values
    return out[:, : a.shape[1]]


def _joint(tabs):
    h = tabs[0]
    for t in tabs[1:]:
        h = _maxmin(h, t)
    return h


def _floor_mask(p, opt, ratio, rate):
    """Options that meet their class's floor, and whether all floors fit."""
    ok = torch.ones_like(ratio, dtype=torch.bool)
    n = ratio.shape[0]
    need, can = torch.zeros(n, dtype=torch.float64, device="cuda"), torch.ones(n, dtype=torch.bool, device="cuda")
    fl = p.floor_rps if p.floor_rps is not None else np.zeros(p.n_classes, np.float32)
    for i in np.flatnonzero(fl > 0):
        cols = torch.from_numpy(np.flatnonzero(opt[:, 0] == i)).cuda()
        ok[:, cols] = (ratio[:, cols] > 0) & (rate[:, cols] >= float(fl[i]))
        cost = torch.from_numpy(opt[opt[:, 0] == i, 3].astype(np.float64)).cuda().expand(n, -1)
        least = torch.where(ok[:, cols], cost, math.inf).amin(1) if len(cols) else torch.full_like(need, math.inf)
        need, can = need + least, can & torch.isfinite(least)
    return ok, can & (need <= p.budget), np.flatnonzero(fl > 0)


def _solve64(p, opt, cap, tail, lex=False):
    """tau*, and the goodput of the chosen allocation (fewest GPUs per class,
    or the largest total for the whole objective)."""
    ratio, rate = _ratios(p, opt, cap, tail)
    ok, met, crit = _floor_mask(p, opt, ratio, rate)
    use = ok | ~met[:, None]
    need = torch.zeros((ratio.shape[0], p.n_classes), dtype=torch.bool, device="cuda")
    for i in crit:  # a class that has to meet its floor can't stay empty
        need[:, i] = met
    masked = torch.where(use, ratio, 0.0)
    if len(crit):
        tabs = _class_tables(p, opt, torch.where(use, ratio, -1.0)).clamp_min(0.0)
        neg = torch.full_like(ratio, -1.0)
        for i in crit:
            cols = torch.from_numpy(np.flatnonzero(opt[:, 0] == i)).cuda()
            t = torch.full((ratio.shape[0], p.budget + 1), -1.0, dtype=torch.float64, device="cuda")
            idx = torch.from_numpy(opt[opt[:, 0] == i, 3]).cuda().expand(ratio.shape[0], -1)
            t.scatter_reduce_(1, idx, torch.where(use, ratio, neg)[:, cols], "amax")
            t = torch.cummax(t, dim=1).values
            tabs[i] = torch.where(met[:, None], t, tabs[i])
    else:
        tabs = _class_tables(p, opt, masked)
    tau = _joint(list(tabs))[:, -1].clamp_min(0.0)
    allowed = use & (ratio >= tau[:, None])
    good = torch.zeros_like(tau)
    if lex:
        layer = torch.zeros((ratio.shape[0], p.budget + 1), dtype=torch.float64, device="cuda")
        for i in range(p.n_classes):
            free = ~need[:, i] & (tau <= 0)
            new = torch.where(free[:, None], layer, -math.inf)
            for q in np.flatnonzero(opt[:, 0] == i):
                cost = int(opt[q, 3])
                v = layer[:, : p.budget + 1 - cost] + torch.where(allowed[:, q], rate[:, q], -math.inf)[:, None]
                new[:, cost:] = torch.maximum(new[:, cost:], v)
            layer = new
        return tau, layer[:, -1]
    for i in range(p.n_classes):
        cols = np.flatnonzero(opt[:, 0] == i)
        if not len(cols):
            continue
        key = torch.from_numpy((opt[cols, 3] * 16 + opt[cols, 1]).astype(np.float64)).cuda()
        at = torch.from_numpy(cols).cuda()
        key = torch.where(allowed[:, at], key[None], math.inf)
        low = key.min(dim=1)
        v = rate[:, at].gather(1, low.indices[:, None])[:, 0]
        empty = ~torch.isfinite(low.values) | ((tau <= 0) & ~need[:, i])
        good = good + torch.where(empty, 0.0, v)
    return tau, good


def _solve64_chunks(p, opt, cap, tail, lex=False):
    step = max(1, int(4e8 // (8 * (3 * len(opt) + 6 * p.n_classes * (p.budget + 1)))))
    got = [_solve64(p, opt, cap[j:j + step], tail[j:j + step], lex) for j in range(0, cap.shape[0], step)]
    return tuple(torch.cat(x) for x in zip(*got))


def _score64(p, iv, cand, cap_s, tail_s):
    """Scores and gaps: of each class the best ratio under each budget and of
    the others jointly, so a sampled cell changes only its own options'."""
    O, E, S = cap_s.shape
    opt = _options(p)
    tau = []
    for cap, tail in ((iv.cap_lo, iv.tail_hi), (iv.cap_hi, iv.tail_lo)):
        ratio, _ = _ratios(p, opt, cap, tail)
        tabs = _class_tables(p, opt, ratio)
        base = _joint(list(tabs))[:, -1]
        val = torch.zeros((O, E, S), dtype=torch.float64, device="cuda")
        for i in sorted({int(x) // (p.n_tp * p.n_levels) for x in cand.tolist()}):
            rest = [tabs[k] for k in range(p.n_classes) if k != i]
            other = _joint(rest) if rest else torch.full((O, p.budget + 1), math.inf, device="cuda").double()
            mine = np.flatnonzero(opt[:, 0] == i)
            for e, x in enumerate(cand.tolist()):
                if x // (p.n_tp * p.n_levels) != i:
                    continue
                on, off = mine[opt[mine, 4] == x], mine[opt[mine, 4] != x]
                at = torch.from_numpy(p.budget - opt[off, 3]).cuda()
                u = torch.minimum(ratio[:, torch.from_numpy(off).cuda()], other[:, at])
                best = u.amax(1) if len(off) else torch.zeros(O, dtype=torch.float64, device="cuda")
                best = best[:, None].expand(O, S)
                ok = tail_s[:, e].double() <= float(p.slo[i])
                for q in on:
                    f = (cap_s[:, e].double() * float(opt[q, 2]) / float(p.demand[i])).clamp_max(1.0)
                    f = torch.minimum(torch.where(ok, f, 0.0), other[:, p.budget - int(opt[q, 3])][:, None])
                    best = torch.maximum(best, f)
                val[:, e] = best
        tau.append((base, val))
    gap = tau[1][0] - tau[0][0]
    score = gap[:, None] - (tau[1][1] - tau[0][1]).mean(2)
    return torch.where(iv.measured[:, cand.long()].bool(), 0.0, score), gap


def _score64_full(p, iv, cand, cap_s, tail_s, lex):
    """Scores and gaps with every scenario's table solved on its own; the
    goodput stage beside the max-min one for the whole objective."""
    O, E, S = cap_s.shape
    opt = _options(p)
    sides = ((iv.cap_lo, iv.tail_hi), (iv.cap_hi, iv.tail_lo))

    def stages(lo, hi):
        top = torch.maximum(lo[1], hi[1])
        return hi[0] - lo[0], torch.where(top > 0, (hi[1] - lo[1]).abs() / top, 0.0)

    now = stages(*(_solve64_chunks(p, opt, *s, lex) for s in sides))
    score = torch.zeros((2, O, E), dtype=torch.float64, device="cuda")
    for o in range(O):
        live = torch.nonzero(iv.measured[o, cand.long()] == 0)[:, 0]
        per = max(1, int(2e8 // (8 * p.n_cells * S)))
        for j in range(0, len(live), per):
            es = live[j:j + per]
            rows, n = torch.arange(len(es) * S, device="cuda"), len(es) * S
            cells = cand[es].long().repeat_interleave(S)
            got = []
            for cap, tail in sides:
                a, b = cap[o].expand(n, -1).clone(), tail[o].expand(n, -1).clone()
                a[rows, cells], b[rows, cells] = cap_s[o, es].reshape(-1), tail_s[o, es].reshape(-1)
                got.append(_solve64_chunks(p, opt, a, b, lex))
            for k, x in enumerate(stages(*got)):
                score[k, o, es] = now[k][o] - x.view(len(es), S).mean(1)
    return score, now


def exact(case, seed):
    c, d = case, _inputs(case, seed)
    p, iv, kind = d["problem"], d["iv"], case["kind"]
    if kind in ("solve", "solve_lex"):
        tau, good = _solve64_chunks(p, _options(p), d["cap"], d["tail"], kind == "solve_lex")
        got = dict(objective=tau, goodput=good, tp_index=None, replicas=None, floors_met=None)
        return dict(got, goodput64=good) if kind == "solve_lex" else got
    if kind == "loop":
        tau, _ = _solve64_chunks(p, _options(p), d["truth_cap"], d["truth_tail"])
        return dict(tau_oracle=tau, tau_truth=None, gpu_seconds=None, final=None, state=None, finished=None,
                    rounds=None, reveals=None)
    E = c["E"] or p.n_cells
    if kind == "score_lex" or c.get("floors"):
        P = sum(c["G"] // int(t) for t in p.tp)
        each = c["K"] * c["G"] * (P if kind == "score_lex" else 16)
        if c["O"] * E * c["S"] * each > 3e11:
            return None
        (mm, gp), (gap, gap_gp) = _score64_full(p, iv, d["cand"], d["cap_s"], d["tail_s"], kind == "score_lex")
        if kind == "score_lex":
            return dict(score_maxmin=mm, score_goodput=gp, gap_maxmin=gap, gap_goodput=gap_gp, best=None)
        return dict(score=mm, gap_now=gap, best=None)
    if c["O"] * E * c["S"] * 8 > 1 << 30:  # two tables of every sample's optimum
        return None
    if kind == "policy":
        lim = torch.from_numpy(d["limit"]).cuda()
        cls = torch.arange(p.n_cells, device="cuda") // (p.n_tp * p.n_levels)
        bad = lambda m, s, k: torch.where((m <= lim[k]).all(-1) & (s >= np.float32(0.99)), 0.0, math.inf)  # noqa: E731
        cells = bad(d["tails"], d["succ"], cls)
        samples = bad(d["metric_s"], d["succ_s"], cls[d["cand"].long()][:, None])
        p0 = Problem(p.tp, p.levels, p.demand, np.zeros(p.n_classes, np.float32), p.budget)
        iv = fs.DeviceIntervals(iv.cap_lo, iv.cap_hi, cells[c["O"]:], cells[: c["O"]], iv.measured)
        score, gap = _score64(p0, iv, d["cand"], d["cap_s"], samples)
        return dict(score=score, gap_now=gap, best=None, cells=cells, samples=samples)
    score, gap = _score64(p, iv, d["cand"], d["cap_s"], d["tail_s"])
    got = dict(score=score, gap_now=gap, best=None)
    if kind == "round":
        opt = _options(p)
        lo, hi = _solve64(p, opt, iv.cap_lo, iv.tail_hi), _solve64(p, opt, iv.cap_hi, iv.tail_lo)
        side = lambda v: dict(objective=v[0], goodput=v[1], tp_index=None, replicas=None, floors_met=None)  # noqa: E731
        got.update(gap=hi[0] - lo[0], state=None, cons=side(lo), opt=side(hi))
    return got
