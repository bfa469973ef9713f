"""The table solver of dense batches (budgets past 64 GPUs, at most 16 classes,
no critical floors) and its limits, against the CPU oracle bit for bit."""
import sys

import numpy as np
import pytest

from test_gpu_parity import assert_alloc_equal, env, gpu_solve  # noqa: F401 (env is a fixture)
from test_gpu_solver_edges import edge_tables
from test_gpu_solver_edges import test_certificate_edges as certificate_edges
from test_gpu_solver_edges import test_dense_lex_solver_edges as lex_edges

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,G,tp,levels", [
    (1, 65, [1, 2, 4, 8], 8), (1, 300, [7], 1), (2, 128, [2, 4, 8], 3), (3, 257, [1, 2], 2), (4, 100, [3, 5, 7, 64], 9),
    (5, 129, [1, 2, 3, 4, 5, 6, 7, 8], 12), (8, 256, [1, 2, 4, 8], 8), (9, 192, [1, 2, 4], 5), (16, 96, [1, 2, 4, 8], 8),
    (16, 1024, [1, 2, 4, 8, 16], 12), (15, 1100, [1, 16], 4),    # one block per CU
    (16, 2300, [2, 8], 3), (16, 2400, [2, 8], 3),               # the largest tables, and past them
    (17, 96, [1, 2, 4, 8], 4), (16, 60, [1, 2, 3, 4, 5, 6, 7, 8], 32),  # 17 classes; 4096 cells at a small budget
])
def test_wide_solver_edges(env, orc, K, G, tp, levels):  # noqa: F811
    p, cap, tail = edge_tables(K, G, tp, levels)
    n = len(cap) if G < 512 else 12
    print(f"[gpu] wide edges K={K} G={G} tp={tp}", file=sys.stderr, flush=True)
    want = [orc.solve(p, cap[j], tail[j]) for j in range(n)]
    rows = np.arange(2048 + 61) % n  # blocks with a second realisation
    g = gpu_solve(env, p, cap[rows], tail[rows])
    for j in list(range(n)) + list(range(2040, 2048 + 61)):
        assert_alloc_equal(p, g, j, want[rows[j]], f"K={K} G={G} tp={tp} row {j}")


@pytest.mark.parametrize("K,G,tp,levels", [(2, 300, [7], 1), (4, 96, [1, 2, 4, 8], 8), (8, 256, [1, 2, 4, 8], 8),
                                           (16, 512, [1, 2, 4, 8, 16], 12), (16, 2400, [2, 8], 3)])
def test_wide_certificate_edges(env, orc, K, G, tp, levels):  # noqa: F811
    certificate_edges(env, orc, K, G, tp, levels)


@pytest.mark.parametrize("K,G,tp,levels", [(1, 200, [1, 3], 2), (3, 257, [1, 2], 2), (4, 100, [3, 5, 7, 64], 9),
                                           (6, 128, [1, 2, 4, 8], 8), (17, 70, [1, 2], 4)])
def test_wide_lex_edges(env, orc, K, G, tp, levels):  # noqa: F811
    """The whole objective past 64 GPUs (undominated costs over several groups
    of 64 budgets)."""
    lex_edges(env, orc, K, G, tp, levels)
