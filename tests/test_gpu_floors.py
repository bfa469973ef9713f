"""Scores with critical floors: the exclusion scorer over both variants of the
objective (floors held, floors ignored) against full solves of every scenario
(scoring kernel 1) and the CPU oracle, bit for bit."""
import sys

import numpy as np
import pytest

from paper_2608_19659_amd.synth import Problem, random_problem
from test_gpu_parity import _random_intervals_and_samples, assert_scores_equal, env, gpu_score  # noqa: F401

pytestmark = pytest.mark.gpu


def _floored(p, shares):
    """p with class i's floor at shares[i] of its demand (0: not critical)."""
    f = (np.resize(np.asarray(shares, np.float32), p.n_classes) * p.demand).astype(np.float32)
    return Problem(p.tp, p.levels, p.demand, p.slo, p.budget, floor_rps=f)


def _inputs(p, S, seed):
    return _random_intervals_and_samples(p, 3, S, seed)


@pytest.mark.parametrize("K,G,tp,levels,S,shares", [
    (1, 16, [1, 2, 4, 8], 3, 64, [0.5]),          # one class: no others' table
    (2, 12, [2, 4, 8], 4, 33, [0.3, 0.0]),        # ragged samples, one critical class
    (3, 24, [1, 2, 4, 8], 5, 256, [0.0, 0.4, 1.0]),  # a floor at the whole demand
    (3, 20, [1, 2, 4], 4, 257, [0.2, 1.5, 0.0]),  # a floor above the demand: never met
    (4, 9, [1, 2, 4, 8], 3, 100, [0.9, 0.9]),     # floors that a few scenarios meet together
    (5, 48, [1, 2, 4, 8], 7, 21, [0.1, 0.0, 0.3]),
    (2, 150, [1, 2], 2, 40, [0.6, 0.0]),          # replica ranges longer than a wavefront
    (6, 90, [1, 3, 5], 6, 5, [0.25, 0.5]),
])
def test_floor_scores_match_full_solves_and_oracle(env, orc, K, G, tp, levels, S, shares):  # noqa: F811
    p = _floored(random_problem(seed=500 + K * G + S, K=K, tp=tp, G=G, n_levels=levels), shares)
    iv, cand, cs, ts = _inputs(p, S, seed=G + S)
    print(f"[gpu] floors K={K} G={G} tp={tp} S={S}", file=sys.stderr, flush=True)
    g = gpu_score(env, p, iv, cand, cs, ts, kernel=0)
    full = gpu_score(env, p, iv, cand, cs, ts, kernel=1)
    for a, b, name in zip(g, full, ("score", "gap_now", "best", "tau_dump")):
        np.testing.assert_array_equal(a, b, err_msg=name)
    pick = np.arange(0, len(cand), max(1, len(cand) // 12))
    g = gpu_score(env, p, iv, cand[pick], np.ascontiguousarray(cs[:, pick]), np.ascontiguousarray(ts[:, pick]), kernel=0)
    assert_scores_equal(g, orc.score(p, iv, cand[pick], cs[:, pick], ts[:, pick], n_threads=8))


def test_floor_scores_many_partials_and_invalid_candidates(env):  # noqa: F811
    """More than 16 partials per tile (the two-kernel finalize), and
    candidates outside [0, N), which score NaN."""
    p = _floored(random_problem(seed=77, K=3, tp=[1, 2, 4], G=18, n_levels=3), [0.3, 0.0, 0.2])
    iv, cand, cs, ts = _inputs(p, 5000, seed=3)
    sel = np.array([0, 5, 9, 13], np.int64)
    cand = cand[sel].copy()
    cand[1], cand[3] = -1, p.n_cells
    cs, ts = np.ascontiguousarray(cs[:, sel]), np.ascontiguousarray(ts[:, sel])
    g = gpu_score(env, p, iv, cand, cs, ts, kernel=0, dump=False)
    full = gpu_score(env, p, iv, cand, cs, ts, kernel=1, dump=False)
    np.testing.assert_array_equal(g[0], full[0])
    np.testing.assert_array_equal(g[2], full[2])
    assert np.isnan(g[0][:, [1, 3]]).all()


def test_floor_scores_with_the_smaller_workspace(env):  # noqa: F811
    """A workspace that holds no table of the exclusion scorer still scores,
    by full solves; a little less is refused."""
    torch, fs, ctx = env
    ctx.set_score_kernel(0)
    p = _floored(random_problem(seed=91, K=3, tp=[1, 2, 4], G=18, n_levels=3), [0.4, 0.0, 0.1])
    plain = Problem(p.tp, p.levels, p.demand, p.slo, p.budget)
    iv, cand, cs, ts = _inputs(p, 48, seed=4)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    args = (fs.DeviceIntervals.from_host(iv, "cuda:0"), t(cand), t(cs), t(ts))
    O, E, S = cs.shape
    n = fs.workspace_size(p, O, E, S)
    want = fs.score_candidates(ctx, p, *args, workspace=torch.empty(n, dtype=torch.uint8, device="cuda"))
    took = None
    for size in range(n - 256, 0, -256):  # the smallest workspace that is accepted
        try:
            r = fs.score_candidates(ctx, p, *args, workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
        except fs.FleetSieveError as e:
            assert e.status == fs.FS_ERR_WORKSPACE_TOO_SMALL
            break
        took = size
        torch.cuda.synchronize()
        np.testing.assert_array_equal(r.score.cpu().numpy(), want.score.cpu().numpy())
    assert took is not None and took < n
    assert fs.workspace_size(plain, O, E, S) > 0
