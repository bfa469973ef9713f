"""The register solver (budgets of at most 64 GPUs, at most 16 classes, no
critical floors) and its limits, against the CPU oracle bit for bit."""
import sys

import numpy as np
import pytest

from paper_2608_19659_amd.synth import Intervals, random_point_tables, random_problem
from test_gpu_lex import assert_lex_equal, gpu_solve_lex
from test_gpu_parity import assert_alloc_equal, env, gpu_solve  # noqa: F401 (env is a fixture)

pytestmark = pytest.mark.gpu


EDGES = [
    (1, 1, [1], 1), (1, 64, [1, 2, 4, 8], 8), (2, 7, [2, 4, 8], 3), (3, 2, [1, 2], 2),  # G below K
    (4, 63, [1, 2, 4, 8], 8), (4, 64, [1, 2, 4, 8], 8), (4, 64, [3, 5, 7, 64], 9),      # N above 128: 144 cells
    (4, 65, [1, 2, 4, 8], 8), (5, 48, [1, 2, 4, 8], 7), (8, 64, [1, 2, 3, 4, 6], 5), (9, 33, [1, 2, 4, 8], 6),
    (16, 64, [1, 2, 4, 8], 8), (16, 64, [1, 2, 3, 4, 5, 6, 7, 8], 12), (16, 15, [1, 4], 4),
    (16, 20, [1, 2, 3, 4, 5, 6, 7, 8], 32),             # 4096 cells: more than its LDS holds
    (17, 64, [1, 2, 4, 8], 4),
]


def edge_tables(K, G, tp, levels):
    """A problem of an edge's sizes and 30 realisations of it, some extreme."""
    p = random_problem(seed=31 * K + G + len(tp), K=K, tp=tp, G=G, n_levels=levels)
    cap, tail = random_point_tables(p, 30, seed=G, cap_range=(0.0, 3.0), tail_range=(5.0, 40.0))
    cap[0], tail[1] = 0.0, 1e9          # nothing to serve with; no cell within its SLO
    cap[2], tail[2] = 2.0 ** 64, 0.0    # every option in full
    cap[3] = np.float32(2.0 ** -64)
    tail[4] = np.inf
    tail[5, ::2] = np.inf
    return p, cap, tail


@pytest.mark.parametrize("K,G,tp,levels", EDGES)
def test_dense_solver_edges(env, orc, K, G, tp, levels):  # noqa: F811
    """Both sides of every limit (budget 64, 4 / 8 / 16 classes, 4 / 8 TP
    degrees, 128 cells), budgets below the class count, and a batch that
    gives wavefronts a second realisation (rows repeat, so each is checked)."""
    p, cap, tail = edge_tables(K, G, tp, levels)
    print(f"[gpu] dense edges K={K} G={G} tp={tp}", file=sys.stderr, flush=True)
    want = [orc.solve(p, cap[j], tail[j]) for j in range(len(cap))]
    rows = np.arange(8192 + 61) % len(cap)
    g = gpu_solve(env, p, cap[rows], tail[rows])
    for j in list(range(len(cap))) + list(range(8180, 8192 + 61)):
        assert_alloc_equal(p, g, j, want[rows[j]], f"K={K} G={G} tp={tp} row {j}")


@pytest.mark.parametrize("K,G,tp,levels", EDGES)
def test_dense_lex_solver_edges(env, orc, K, G, tp, levels):  # noqa: F811
    """The same limits under the whole objective."""
    p, cap, tail = edge_tables(K, G, tp, levels)
    print(f"[gpu] dense lex edges K={K} G={G} tp={tp}", file=sys.stderr, flush=True)
    want = [orc.solve(p, cap[j], tail[j], method="lex") for j in range(len(cap))]
    rows = np.arange(8192 + 61) % len(cap)
    g = gpu_solve_lex(env, p, cap[rows], tail[rows])
    for j in list(range(len(cap))) + list(range(8180, 8192 + 61)):
        assert_lex_equal(p, g, j, want[rows[j]], f"K={K} G={G} tp={tp} row {j}")


@pytest.mark.parametrize("K,G,tp,levels", [c for c in EDGES if c[0] > 1])
def test_certificate_edges(env, orc, K, G, tp, levels):  # noqa: F811
    """The same limits for the certificate: states (a measured and a missing
    committed cell among them), gaps and both allocations."""
    torch, fs, ctx = env
    p, cap, tail = edge_tables(K, G, tp, levels)
    rng = np.random.default_rng(K + G)
    hi = np.minimum(cap * rng.choice([1.0, 1.25], cap.shape), 2.0 ** 64).astype(np.float32)
    tlo = np.where(np.isfinite(tail), tail * rng.choice([1.0, 0.5], tail.shape), tail).astype(np.float32)
    meas = np.ones(cap.shape, np.uint8)
    meas[::2] = rng.random(cap[::2].shape) < 0.7
    iv = Intervals(cap, hi, tlo, tail, meas)
    print(f"[gpu] certificate edges K={K} G={G} tp={tp}", file=sys.stderr, flush=True)
    r = fs.certify(ctx, p, fs.DeviceIntervals.from_host(iv, "cuda:0"), eps=0.2)
    torch.cuda.synchronize()
    o = orc.certify(p, iv, eps=0.2)
    np.testing.assert_array_equal(r.state.cpu().numpy(), o.state)
    np.testing.assert_array_equal(r.gap.cpu().numpy(), o.gap)
    cons, opt = ({k: v.cpu().numpy() for k, v in d.items()} for d in (r.cons, r.opt))
    for j in range(len(cap)):
        assert_alloc_equal(p, cons, j, o.cons[j], f"cons {j}")
        assert_alloc_equal(p, opt, j, o.opt[j], f"opt {j}")
