"""Workspaces of callers that keep the size they once asked for: what the
library asked for before it scored problems with critical floors by tables and
before its loops kept refitted candidate intervals still serves every call, with
the same results."""
import sys

import numpy as np
import pytest
import torch  # noqa: F401 (its HIP runtime is the one to load first)

from paper_2608_19659_amd import fleetsieve as fs
from paper_2608_19659_amd.synth import Problem, random_problem
from test_gpu_parity import _random_intervals_and_samples, env  # noqa: F401 (env is a fixture)

# K, G, TP degrees, levels, orders, candidates, samples, critical floors, then the sizes of that time: the score, the
# stage-wise score, the loop, the loop with refit
FORMER = [
    (3, 18, [1, 2, 4], 3, 3, 27, 48, 1, 11776, 13056, 20736, 53504),
    (3, 18, [1, 2, 4], 3, 3, 27, 48, 0, 17920, 341248, 348928, 381696),
    (2, 70, [1, 2, 4, 8], 6, 4, 48, 16, 1, 20736, 22784, 33024, 59904),
    (2, 16, [1, 2, 4, 8], 3, 2, 24, 1, 0, 12288, 100096, 106240, 107520),  # one sample: no room in the clamped copies
    (5, 48, [1, 2, 4, 8], 7, 12, 140, 999, 1, 341248, 556800, 617216, 14064640),
    (4, 64, [1, 2, 4, 8], 8, 16, 128, 64, 0, 448512, 34706432, 34777856, 35851008),
]


def _problem(K, G, tp, levels, critical):
    p = random_problem(seed=K * G, K=K, tp=tp, G=G, n_levels=levels)
    if critical:
        p = Problem(p.tp, p.levels, p.demand, p.slo, p.budget, floor_rps=(0.25 * p.demand).astype(np.float32))
    return p


@pytest.mark.parametrize("case", FORMER, ids=lambda c: f"{c[0]}x{c[1]}-{c[7]}")
def test_sizes_did_not_grow_where_no_table_was_added(case):
    K, G, tp, levels, O, E, S, critical, score, lex, loop, refit = case
    p = _problem(K, G, tp, levels, critical)
    assert fs.score_lex_workspace_size(p, O, E, S) <= lex
    if not critical:  # (with floors the tables come on top, and may be left out)
        assert fs.workspace_size(p, O, E, S) <= score
        assert fs.loop_workspace_size(p, O, E, S) <= loop
        assert fs.loop_refit_workspace_size(p, O, E, S) <= refit


def _host(r):
    out = {}
    for k, v in vars(r).items():
        if v is None:
            continue
        for name, x in (v.items() if isinstance(v, dict) else [("", v)]):
            out[k + name] = x.cpu().numpy()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("lex", [0, 1])
@pytest.mark.parametrize("case", FORMER[:4], ids=lambda c: f"{c[0]}x{c[1]}-{c[7]}")
def test_calls_with_the_former_sizes(env, case, lex):  # noqa: F811
    _, _, ctx = env
    K, G, tp, levels, O, E, S, critical, score, lex_size, loop, refit = case
    p = _problem(K, G, tp, levels, critical)
    iv, cand, cs, ts = _random_intervals_and_samples(p, O, S, seed=G)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    d = fs.DeviceIntervals.from_host(iv, "cuda:0")
    dc, dcs, dts = t(cand), t(cs), t(ts)
    tc, tt = t((iv.cap_lo + iv.cap_hi) * np.float32(0.5)), t((iv.tail_lo + iv.tail_hi) * np.float32(0.5))
    calls = []
    if lex:
        calls.append(("stage-wise score", lex_size, lambda ws: fs.score_candidates_lex(ctx, p, d, dc, dcs, dts, workspace=ws)))
    else:
        calls.append(("score", score, lambda ws: fs.score_candidates(ctx, p, d, dc, dcs, dts, workspace=ws)))
    for r, size in ((False, loop), (True, refit)):
        calls.append((f"loop refit={r}", size, lambda ws, r=r: fs.profile_loop(
            ctx, p, d, tc, tt, dc, dcs, dts, eps=0.01, max_rounds=5, workspace=ws, refit=r)))
    ctx.set_option(fs.OPT_LOOP_OBJECTIVE, lex)
    try:
        for name, size, call in calls:
            print(f"[gpu] former workspace {name} K={K} G={G} critical={critical} lex={lex}", file=sys.stderr, flush=True)
            want = _host(call(None))
            buf = torch.full((size + (1 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
            got = _host(call(buf[:size]))
            torch.cuda.synchronize()
            assert bool((buf[size:] == 0xA5).all()), f"{name}: written past the workspace"
            for k in want:
                np.testing.assert_array_equal(got[k], want[k], err_msg=f"{name} {k}")
    finally:
        ctx.set_option(fs.OPT_LOOP_OBJECTIVE, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("E", [24, 5000, 16384])
def test_fixed_order_loops_keep_no_candidate_intervals(env, E):  # noqa: F811
    """A refitting loop with a fixed reveal order has no samples, so its
    workspace has no room for the scorer's copy of the candidates' intervals
    (16 bytes each; the candidates repeat): nothing is written past it, and the
    loop is the general path's."""
    _, _, ctx = env
    p = _problem(2, 16, [1, 2, 4, 8], 3, 0)
    iv, cells, cs, ts = _random_intervals_and_samples(p, 2, 1, seed=5)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rng = np.random.default_rng(E)
    order = t(np.stack([rng.permutation(E) for _ in range(2)]).astype(np.int32))
    d, cand = fs.DeviceIntervals.from_host(iv, "cuda:0"), t(np.resize(cells, E))
    tc, tt = t((iv.cap_lo + iv.cap_hi) * np.float32(0.5)), t((iv.tail_lo + iv.tail_hi) * np.float32(0.5))
    call = lambda ws: _host(fs.profile_loop(  # noqa: E731
        ctx, p, d, tc, tt, cand, t(cs), t(ts), eps=-1.0, policy=fs.POLICY_ORDER, order=order, max_rounds=30, workspace=ws,
        refit=True))
    size = fs.loop_refit_workspace_size(p, 2, E, 0)
    print(f"[gpu] fixed-order refit loop E={E} workspace={size}", file=sys.stderr, flush=True)
    buf = torch.full((size + (1 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
    got = call(buf[:size])
    torch.cuda.synchronize()
    assert bool((buf[size:] == 0xA5).all()), "written past the workspace"
    ctx.set_score_kernel(1)
    try:
        want = call(None)
    finally:
        ctx.set_score_kernel(0)
    for k in want:
        np.testing.assert_array_equal(got[k], want[k], err_msg=k)
