"""Stage-wise score where the replica counts a scenario can use differ widely
between lanes: cells that serve the whole demand with one replica or with
none, tails that break the SLO everywhere, demand far below and far above the
capacity."""
import sys
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from paper_2608_19659_amd.synth import random_problem
from test_gpu_lex import _assert_score_lex_equal, _random_score_inputs, _score_lex, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G", [7, 63, 64, 65, 130])  # one cost per lane up to 64
@pytest.mark.parametrize("scale", [0.02, 1.0, 40.0])
def test_counts_that_matter(env, G, scale):  # noqa: F811
    p = random_problem(seed=7300 + G, K=3, tp=[1, 2, 3, 4, 8][:4 + G % 2], G=G, n_levels=4)
    iv, cand, cs, ts = _random_score_inputs(p, 2, 70, seed=G)
    rng = np.random.default_rng(G)
    kind = rng.integers(0, 4, iv.cap_lo.shape)
    f = np.where(kind == 1, 0.0, np.where(kind == 2, scale, 1.0)).astype(np.float32)
    iv.cap_lo[:], iv.cap_hi[:] = iv.cap_lo * f, iv.cap_hi * f
    cs = (cs * f[:, :, None]).astype(np.float32)
    bad = np.float32(1e6)
    iv.tail_lo[kind == 3] = iv.tail_hi[kind == 3] = bad
    ts[kind == 3] = bad
    print(f"[gpu] stage-wise counts G={G} scale={scale}", file=sys.stderr, flush=True)
    g = _score_lex(env, SimpleNamespace(problem=p, intervals=iv, cand=cand), cs, ts)
    o = oracle.score_lex(p, iv, cand, cs, ts, n_threads=8)
    _assert_score_lex_equal(g, o, f"G={G} scale={scale}")
