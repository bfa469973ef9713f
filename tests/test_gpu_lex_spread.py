"""The whole objective where served rates lie so far apart that binary64 sums
absorb the small ones: allocations whose totals tie only through rounding go
to the fewest GPUs, as in the oracle, so no cost may be left out of the
knapsack.  One TP degree of 1 (one option per cost), a load level per replica
count as far as the levels go."""
import sys

import numpy as np
import pytest

from paper_2608_19659_amd.synth import Intervals, Problem
from test_gpu_lex import assert_lex_equal, env, gpu_solve_lex  # noqa: F401 (env is a fixture)
from test_gpu_parity import assert_alloc_equal

pytestmark = pytest.mark.gpu

SIZES = [(2, 5, 0), (3, 9, 0), (4, 33, 0), (8, 64, 0), (1, 12, 0),  # in registers
         (3, 70, 0), (5, 140, 0), (17, 24, 0),                     # in LDS
         (3, 9, 1), (4, 20, 1)]                                     # a critical class
DEMAND = np.float32(2.0 ** 32)


def spread_problem(K, G, critical, demand=DEMAND):
    n = min(G, 32)
    d = np.full(K, demand, np.float32)
    d[1:] *= np.float32(0.75)  # other loads per replica, other cells
    floor = None
    if critical:
        floor = np.zeros(K, np.float32)
        floor[K // 2] = np.float32(2.0 ** -31)
    return Problem(tp=[1], levels=sorted(demand / np.float32(r) for r in range(1, n + 1)), demand=d, slo=np.full(K, 30.0),
                   budget=G, floor_rps=floor)


def spread_tables(p, n, seed):
    """Every class of a realisation has rates of one magnitude -- the demand
    (met by several costs), about 1, about 2^-31 -- of few distinct values; the
    first rows have ordinary rates."""
    rng = np.random.default_rng(seed)
    K, B = p.n_classes, p.n_levels
    mag = rng.choice([32.0, 32.0, 0.0, -31.0, -31.0], (n, K, 1))
    r = np.exp2(mag) * rng.choice([0.0, 0.25, 0.5, 1.0, 1.0, 2.0], (n, K, B))
    r[: n // 8] = rng.choice([0.0, 0.5, 1.0, 1.5], (n // 8, K, B))
    tail = np.where(rng.random((n, K, B)) < 0.15, 50.0, 10.0)
    return r.reshape(n, K * B).astype(np.float32), tail.reshape(n, K * B).astype(np.float32)


@pytest.mark.parametrize("K,G,critical", SIZES)
def test_dense_solves(env, orc, K, G, critical):  # noqa: F811
    p = spread_problem(K, G, critical)
    cap, tail = spread_tables(p, 300 if G < 100 else 100, seed=K * G)
    print(f"[gpu] spread rates K={K} G={G} critical={critical}", file=sys.stderr, flush=True)
    g = gpu_solve_lex(env, p, cap, tail)
    for j in range(len(cap)):
        assert_lex_equal(p, g, j, orc.solve(p, cap[j], tail[j], "lex"), f"row {j}")


@pytest.mark.parametrize("K,G,critical", [(3, 9, 0), (3, 70, 0), (3, 9, 1)])
def test_certificates(env, orc, K, G, critical):  # noqa: F811
    torch, fs, ctx = env
    p = spread_problem(K, G, critical)
    cap, tail = spread_tables(p, 200, seed=K + G)
    rng = np.random.default_rng(G)
    hi = np.where(rng.random(cap.shape) < 0.5, cap, cap * 2).astype(np.float32)
    iv = Intervals(cap, hi, tail, tail, (rng.random(cap.shape) < 0.8).astype(np.uint8))
    print(f"[gpu] spread certificates K={K} G={G} critical={critical}", file=sys.stderr, flush=True)
    r = fs.certify_lex(ctx, p, fs.DeviceIntervals.from_host(iv, "cuda:0"), eps=0.2)
    torch.cuda.synchronize()
    o = orc.certify_lex(p, iv, 0.2)
    np.testing.assert_array_equal(r.state.cpu().numpy(), o.state)
    np.testing.assert_array_equal(r.gap_goodput.cpu().numpy(), o.gap_gp)
    for name, got, want in (("cons", r.cons, o.cons), ("opt", r.opt, o.opt)):
        got = {k: v.cpu().numpy() for k, v in got.items()}
        for j in range(len(cap)):
            assert_alloc_equal(p, got, j, want[j], f"{name} {j}")


@pytest.mark.parametrize("G", [9, 70])
def test_demands_far_apart(env, orc, G):  # noqa: F811
    """A demand 2^40 below the largest: served rates that far apart whatever the
    capacities."""
    p = spread_problem(3, G, 0)
    p = Problem(p.tp, p.levels, np.array([p.demand[0], 2.0 ** -8, p.demand[2]], np.float32), p.slo, p.budget)
    rng = np.random.default_rng(G)
    cap = (2.0 ** 31 * rng.choice([0.0, 0.25, 0.5, 1.0], (120, p.n_cells))).astype(np.float32)
    tail = np.full(cap.shape, 10.0, np.float32)
    print(f"[gpu] demands far apart G={G}", file=sys.stderr, flush=True)
    g = gpu_solve_lex(env, p, cap, tail)
    for j in range(len(cap)):
        assert_lex_equal(p, g, j, orc.solve(p, cap[j], tail[j], "lex"), f"row {j}")
