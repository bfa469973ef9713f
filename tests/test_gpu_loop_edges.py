"""The profiling loop where its paths differ: the launches of three kernels a
round (no critical floors, budgets of at most 64 GPUs, at most 16 classes,
the max-min objective) and the general ones, against the loop oracle."""
import sys

import numpy as np
import pytest

import oracle
from paper_2608_19659_amd.synth import Intervals, Problem
from test_gpu_loop import _inputs, assert_loop_equal, env, gpu_loop  # noqa: F401 (env is a fixture)

pytestmark = pytest.mark.gpu


def note(msg):
    print(f"[gpu] {msg}", file=sys.stderr, flush=True)


@pytest.mark.parametrize("budget,floors,kernel,lex", [
    (16, None, 0, 0), (16, None, 1, 0),  # three launches a round; the general ones
    (16, [0.5, 0.0], 0, 0), (70, None, 0, 0), (16, None, 0, 1), (70, None, 0, 1),
])
def test_a_class_without_a_tail_limit(env, budget, floors, kernel, lex):  # noqa: F811
    """An SLO of +inf: an undecided trajectory still returns an allocation of
    measured cells only."""
    torch, fs, ctx = env
    w, p, tc, tt, cs, ts = _inputs("paper-shaped-2class-G16", list(range(6)), 8)
    p = Problem(p.tp, p.levels, p.demand, np.array([np.inf, np.inf], np.float32), budget,
                floor_rps=None if floors is None else np.asarray(floors, np.float32))
    note(f"loop without tail limits G={budget} floors={floors} kernel={kernel} lex={lex}")
    o = oracle.profile_loop(p, w.intervals, tc, tt, w.cand, cs, ts, eps=-1.0, max_rounds=2, n_threads=8,
                            objective="lex" if lex else "maxmin")
    ctx.set_score_kernel(kernel)
    ctx.set_option(fs.OPT_LOOP_OBJECTIVE, lex)
    try:
        g = gpu_loop(env, p, w.intervals, tc, tt, w.cand, cs, ts, -1.0, 0, max_rounds=2)
    finally:
        ctx.set_score_kernel(0)
        ctx.set_option(fs.OPT_LOOP_OBJECTIVE, 0)
    assert_loop_equal(g, o, f"G={budget} floors={floors} kernel={kernel} lex={lex}")


@pytest.mark.parametrize("floors", [None, [1.0, 0.0]])
def test_progress_checks_are_refused_under_capture(env, floors):  # noqa: F811
    """check_every > 0 waits for the stream, which a capture cannot: refused
    before anything is enqueued, so the capture goes on; check_every = 0, and
    checks that no round reaches, are captured.  Afterwards the context's loops
    are what they were."""
    torch, fs, ctx = env
    w, p, tc, tt, cs, ts = _inputs("paper-shaped-2class-G16", [0, 1, 2], 16, floors=floors)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    args = (fs.DeviceIntervals.from_host(w.intervals, "cuda:0"), t(tc), t(tt), t(w.cand), t(cs), t(ts))
    call = lambda n: fs.profile_loop(ctx, p, *args, eps=0.05, max_rounds=8, check_every=n)  # noqa: E731
    want = call(1)
    torch.cuda.synchronize()
    note(f"loop under capture floors={floors}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        with pytest.raises(fs.FleetSieveError) as e:
            call(1)
        got = call(0)
        late = call(8)
    assert e.value.status == fs.FS_ERR_DEVICE
    for _ in range(3):
        for x in (got.state, got.rounds, got.reveals, got.tau_truth):
            x.zero_()
        graph.replay()
        eager = call(1)
        torch.cuda.synchronize()
        for k in ("state", "rounds", "reveals", "tau_truth", "gpu_seconds"):
            assert torch.equal(getattr(got, k), getattr(want, k)), k
            assert torch.equal(getattr(late, k), getattr(want, k)), k
            assert torch.equal(getattr(eager, k), getattr(want, k)), k


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_samples_at_any_float(env, offset):  # noqa: F811
    """Sample arrays that start 4, 8 or 12 bytes past a 16-byte boundary (a
    multiple of 4 samples, read four at a time), in the score and in loops
    that clamp them as they are read."""
    torch, fs, ctx = env
    w, p, tc, tt, cs, ts = _inputs("paper-shaped-2class-G16", [0, 1, 2, 3], 32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731

    def shifted(a):
        buf = torch.empty(a.size + offset, dtype=torch.float32, device="cuda")
        v = buf[offset:].view(a.shape)
        v.copy_(t(a))
        assert v.data_ptr() % 16 == 4 * offset
        return v

    d, dc, dtc, dtt = fs.DeviceIntervals.from_host(w.intervals, "cuda:0"), t(w.cand), t(tc), t(tt)
    note(f"samples {4 * offset} bytes past a boundary")
    a, b = (fs.score_candidates(ctx, p, d, dc, x, y) for x, y in ((t(cs), t(ts)), (shifted(cs), shifted(ts))))
    torch.cuda.synchronize()
    assert torch.equal(a.score, b.score) and torch.equal(a.best, b.best)
    for refit in (False, True):
        a, b = (fs.profile_loop(ctx, p, d, dtc, dtt, dc, x, y, eps=0.05, max_rounds=6, refit=refit)
                for x, y in ((t(cs), t(ts)), (shifted(cs), shifted(ts))))
        torch.cuda.synchronize()
        for k in ("state", "rounds", "reveals", "tau_truth"):
            assert torch.equal(getattr(a, k), getattr(b, k)), (refit, k)


TP4, TP5, TP8 = [1, 2, 4, 8], [1, 2, 3, 4, 6], [1, 2, 3, 4, 5, 6, 7, 8]

# K, G, TP degrees, levels, candidates, samples, rounds, refit
ROUNDS = [
    # more than 16 partials a tile: the pick is the finalize's
    (2, 16, TP4, 3, 5, 8196, 2, False), (2, 16, TP4, 3, 5, 8193, 2, True),
    # one, two, five and six scoring wavefronts, the last with a second turn
    (2, 16, TP4, 3, 128, 4, 6, False), (2, 16, TP4, 3, 129, 4, 6, True), (2, 16, TP4, 3, 600, 3, 6, False),
    (2, 16, TP4, 3, 900, 3, 6, True),
    # samples clamped as they are read, one at a time and four at a time
    (4, 64, TP4, 4, 64, 33, 8, True), (4, 64, TP4, 4, 64, 36, 8, True),
    # the class and TP counts the kernels are compiled for, at their limits
    (4, 30, TP5, 3, 60, 6, 8, True), (4, 30, TP8, 3, 96, 6, 8, False), (5, 31, TP4, 3, 60, 6, 8, True),
    (8, 64, TP4, 3, 96, 6, 8, False), (8, 40, TP8, 2, 128, 5, 6, True), (9, 37, TP4, 3, 108, 6, 6, True),
    (16, 64, TP4, 2, 128, 5, 6, True), (12, 64, TP5, 2, 120, 5, 6, False), (16, 64, TP8, 2, 256, 4, 4, True),
]


def rounds_case(K, G, tp, levels, E, S, seed):
    """Six trajectories (a third of the cells measured) of a problem whose
    classes want about half of what G / K GPUs serve each, E candidates (cells,
    repeated if there are fewer), samples and a truth inside the intervals."""
    rng = np.random.default_rng(seed)
    O, n_tp = 6, len(tp)
    demand = (0.5 * G / K * rng.uniform(0.6, 1.4, K)).astype(np.float32)
    p = Problem(tp=tp, levels=demand.max() * np.float32(0.5) ** np.arange(levels - 1, -1, -1, dtype=np.float32),
                demand=demand, slo=np.full(K, 30.0, np.float32), budget=G)
    shape = (O, K, n_tp, levels)
    mid = rng.uniform(0.5, 1.1, shape) * np.asarray(tp)[:, None]
    tail = rng.uniform(10.0, 32.0, shape)
    meas = (rng.random((O, p.n_cells)) < 0.33).astype(np.uint8)
    width = np.where(meas.reshape(shape) != 0, 0.0, rng.uniform(0.05, 0.6, shape))
    flat = lambda a: np.ascontiguousarray(a.reshape(O, -1).astype(np.float32))  # noqa: E731
    iv = Intervals(flat(mid * (1 - width)), flat(mid * (1 + width)), flat(tail * (1 - 0.5 * width)),
                   flat(tail * (1 + 0.5 * width)), meas)
    cand = np.resize(rng.permutation(p.n_cells), E).astype(np.int32)
    inside = lambda lo, hi, u: (lo + (hi - lo) * u.astype(np.float32)).astype(np.float32)  # noqa: E731
    u, v = rng.random((2, O, E, S)), rng.random((2, O, p.n_cells))
    cs = inside(iv.cap_lo[:, cand, None], iv.cap_hi[:, cand, None], u[0])
    ts = inside(iv.tail_lo[:, cand, None], iv.tail_hi[:, cand, None], u[1])
    return p, iv, cand, cs, ts, inside(iv.cap_lo, iv.cap_hi, v[0]), inside(iv.tail_lo, iv.tail_hi, v[1])


@pytest.mark.parametrize("case", ROUNDS, ids=lambda c: f"{c[0]}x{c[1]}-tp{len(c[2])}-E{c[4]}-S{c[5]}-refit{int(c[7])}")
def test_rounds_of_three_launches(env, case, monkeypatch):  # noqa: F811
    """Every way a round picks, clamps and is compiled, against the oracle."""
    torch, fs, ctx = env
    K, G, tp, levels, E, S, rounds, refit = case
    p, iv, cand, cs, ts, tc, tt = rounds_case(K, G, tp, levels, E, S, seed=100 + K * G + E)
    note(f"loop rounds K={K} G={G} tp={tp} E={E} S={S} refit={refit}")
    o = oracle.profile_loop(p, iv, tc, tt, cand, cs, ts, eps=0.0, max_rounds=rounds, n_threads=8, refit=refit)
    assert (o.rounds > 1).any()  # picks that follow a reveal
    loop = fs.profile_loop
    monkeypatch.setattr(fs, "profile_loop", lambda *a, **k: loop(*a, refit=refit, **k))
    assert_loop_equal(gpu_loop(env, p, iv, tc, tt, cand, cs, ts, 0.0, 0, max_rounds=rounds), o, str(case))
