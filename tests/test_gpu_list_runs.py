"""The exclusion scorer's work list in several runs of orders: the same scores
as full re-solves (the lane kernel), whatever the runs and the grid; runs of
unequal lengths, and few orders with many candidates."""
import sys

import numpy as np
import pytest

from paper_2608_19659_amd.synth import Intervals, make_workload
from test_gpu_parity import env, gpu_score  # noqa: F401

pytestmark = pytest.mark.gpu


def _agree(env, O, E, setup, waves, S=20):  # noqa: F811
    """E candidates: the workload's 48 cells, repeated."""
    torch, fs, ctx = env
    w = make_workload("paper-shaped-2class-G16", orders=list(range(min(O, 200))), with_samples=False)
    if O > 200:  # the orders repeat
        w.intervals = Intervals(*(np.resize(a, (O, a.shape[1])) for a in vars(w.intervals).values()))
    cand = np.resize(w.cand, E)
    rng = np.random.default_rng(O)
    lo, hi = w.intervals.cap_lo[:, cand, None], w.intervals.cap_hi[:, cand, None]
    tl, th = w.intervals.tail_lo[:, cand, None], w.intervals.tail_hi[:, cand, None]
    shape = (O, E, S)
    cs = (lo + (hi - lo) * rng.random(shape)).astype(np.float32)
    ts = (tl + (th - tl) * rng.random(shape)).astype(np.float32)
    print(f"[gpu] list runs O={O} E={E} setup={setup} waves={waves}", file=sys.stderr, flush=True)
    ctx.set_option(fs.OPT_SETUP, setup)
    ctx.set_option(fs.OPT_SCORER_WAVES, waves)
    try:
        g = gpu_score(env, w.problem, w.intervals, cand, cs, ts, kernel=3)
    finally:
        ctx.set_option(fs.OPT_SETUP, 0)
        ctx.set_option(fs.OPT_SCORER_WAVES, 0)
    full = gpu_score(env, w.problem, w.intervals, cand, cs, ts, kernel=2)
    for a, b, name in zip(g, full, ("score", "gap_now", "best", "tau_dump")):
        np.testing.assert_array_equal(a, b, err_msg=name)


@pytest.mark.parametrize("O", [25, 26, 51, 101, 150, 200])  # 1 (1,200 tiles), 2, 4, 8, and runs that do not divide O
@pytest.mark.parametrize("setup,waves", [(0, 0), (0, 1), (0, 3), (0, 513), (0, 2500), (1, 0), (1, 5)])  # blocks of 1, 2, 5, 8 wavefronts
def test_list_runs_agree_with_full_solves(env, O, setup, waves):  # noqa: F811
    _agree(env, O, 48, setup, waves)


@pytest.mark.parametrize("O,E", [(3, 1300), (5, 2000), (9, 1152), (12, 1000), (17, 600)])  # 2, 4, 8, 8, 8 runs
@pytest.mark.parametrize("setup,waves", [(0, 0), (0, 5), (1, 0)])
def test_few_orders_with_many_candidates(env, O, E, setup, waves):  # noqa: F811
    _agree(env, O, E, setup, waves)


@pytest.mark.parametrize("O,E", [(1300, 48), (1300, 3), (3400, 48), (3400, 2), (28000, 2)])
@pytest.mark.parametrize("setup", [0, 1])
def test_many_orders(env, O, E, setup):  # noqa: F811
    """Revealed flags of all orders past what a list block stages (60 KB beside
    the per-order set-up, 156 KB beside the general one): more runs than the
    tiles ask for, and at 28,000 orders the list from global memory."""
    _agree(env, O, E, setup, 0, S=4)
