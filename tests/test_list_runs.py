"""The exclusion scorer's work list in runs of orders (csrc/fs_list.h): the
runs of a call cover its orders, every run has one, so that no thread of the
scorer takes its first entry from past the list, and their number follows from
what a block can stage of one run."""
import ctypes
import os
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2608_19659_amd", "csrc")
SHIM = """
#include "fs_list.h"
extern "C" void runs_of(int O, long most, int *out, int *first) {
  const fs::ListRuns r = fs::list_runs_of(O, most);
  out[0] = r.log; out[1] = r.n; out[2] = r.O; out[3] = r.per;
  for (int q = 0; q <= r.n; ++q) first[q] = r.first(q);
}
extern "C" int staged(int O, long want, long most, int longest) {
  fs::ListRuns r{};
  const bool ok = fs::list_runs_staged(O, want, most, [&](int per) { return per <= longest; }, &r);
  return ok ? r.n : 0;
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("runs")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "libshim.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


@pytest.fixture(scope="module")
def runs_of(shim):
    def call(O, most):
        out, first = (ctypes.c_int * 4)(), (ctypes.c_int * 65)()
        shim.runs_of(O, ctypes.c_long(most), out, first)
        log, n, orders, per = out
        assert n == 1 << log and orders == O
        return n, per, list(first[: n + 1])

    return call


@pytest.mark.parametrize("most", range(1, 9))
def test_every_run_has_an_order(runs_of, most):
    for O in [*range(1, 300), 999, 4095, 65533, 65535]:
        n, per, first = runs_of(O, most)
        assert 1 <= n <= min(most, O) and 2 * n > min(most, O), (O, most)
        assert first[0] == 0 and first[n] == O, (O, most, first)
        lengths = [b - a for a, b in zip(first, first[1:])]
        assert min(lengths) >= 1 and max(lengths) == per, (O, most, first)


def test_runs_are_sized_by_what_one_stages(shim, runs_of):
    """As many runs as wanted, or more until the longest can be staged, never
    none where that is possible."""
    for O in (1, 2, 5, 9, 64, 200, 3400):
        for want in (1, 2, 8):
            for longest in (1, 2, 3, 25, 200, 425, 4000):
                n = shim.staged(O, ctypes.c_long(want), ctypes.c_long(8), longest)
                sizes = [m for m in (1, 2, 4, 8) if m <= O]
                least = max(m for m in sizes if m <= want)
                fit = [m for m in sizes if m >= least and runs_of(O, m)[1] <= longest]
                assert n == (fit[0] if fit else 0), (O, want, longest)
