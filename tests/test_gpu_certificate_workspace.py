"""The certificates within their workspace: records of as many orders as it
holds at a time, nothing written past it, the same results whatever its size."""
import sys

import numpy as np
import pytest

from paper_2608_19659_amd.synth import Intervals, random_point_tables, random_problem
from test_gpu_parity import assert_alloc_equal, env  # noqa: F401 (env is a fixture)

pytestmark = pytest.mark.gpu

# in registers; by tables in LDS; with critical floors; past 16 classes
SIZES = [(3, 9, False), (4, 96, False), (3, 20, True), (17, 24, False)]
GUARD = 0xA5


def _intervals(p, O, seed):
    cap, tail = random_point_tables(p, O, seed=seed, cap_range=(0.0, 3.0), tail_range=(5.0, 40.0))
    rng = np.random.default_rng(seed)
    hi = (cap * rng.choice([1.0, 1.25], cap.shape)).astype(np.float32)
    return Intervals(cap, hi, (tail * rng.choice([1.0, 0.5], tail.shape)).astype(np.float32), tail,
                     (rng.random(cap.shape) < 0.8).astype(np.uint8))


@pytest.mark.parametrize("lex", [False, True])
@pytest.mark.parametrize("K,G,critical", SIZES)
def test_certificates_stay_in_their_workspace(env, orc, K, G, critical, lex):  # noqa: F811
    torch, fs, ctx = env
    p = random_problem(seed=77 + K + G, K=K, tp=[1, 2, 4], G=G, n_levels=4, critical=critical)
    O = 37
    iv = _intervals(p, O, seed=G)
    d = fs.DeviceIntervals.from_host(iv, "cuda:0")
    call = fs.certify_lex if lex else fs.certify
    want = (orc.certify_lex if lex else orc.certify)(p, iv, 0.2)
    # the layout without orders holds one order's records; 5 and all 37
    for n in (fs.workspace_size(p), fs.workspace_size(p, 5), fs.workspace_size(p, O)):
        print(f"[gpu] certificate workspace K={K} G={G} critical={critical} lex={lex} bytes={n}", file=sys.stderr,
              flush=True)
        # (room for every order's records behind it, so that a stray write stays in the allocation)
        buf = torch.full((n + (1 << 20),), GUARD, dtype=torch.uint8, device="cuda")
        r = call(ctx, p, d, eps=0.2, workspace=buf[:n])
        torch.cuda.synchronize()
        assert bool((buf[n:] == GUARD).all()), "written past the workspace"
        np.testing.assert_array_equal(r.state.cpu().numpy(), want.state)
        if lex:
            np.testing.assert_array_equal(r.gap_maxmin.cpu().numpy(), want.gap_mm)
            np.testing.assert_array_equal(r.gap_goodput.cpu().numpy(), want.gap_gp)
        else:
            np.testing.assert_array_equal(r.gap.cpu().numpy(), want.gap)
        for name, got, ref in (("cons", r.cons, want.cons), ("opt", r.opt, want.opt)):
            got = {k: v.cpu().numpy() for k, v in got.items()}
            for j in range(O):
                assert_alloc_equal(p, got, j, ref[j], f"{name} {j}")


def test_binding_asks_for_every_order(env):  # noqa: F811
    """Without a workspace argument the context's buffer holds all records."""
    torch, fs, _ = env
    p = random_problem(seed=5, K=3, tp=[1, 2, 4], G=20, n_levels=4, critical=True)
    ctx = fs.Context(0)
    O = 64
    fs.certify_lex(ctx, p, fs.DeviceIntervals.from_host(_intervals(p, O, 3), "cuda:0"), eps=0.2)
    torch.cuda.synchronize()
    assert ctx.workspace(1).numel() >= fs.workspace_size(p, O)
    ctx.close()
