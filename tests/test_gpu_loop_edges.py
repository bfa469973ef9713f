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
