"""The profiling loop where its paths differ: the launches of three kernels a
round (no critical floors, budgets of at most 64 GPUs, at most 16 classes,
the max-min objective) and the general ones, against the loop oracle."""
import sys

import numpy as np
import pytest

import oracle
from paper_2608_19659_amd.synth import Problem
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
