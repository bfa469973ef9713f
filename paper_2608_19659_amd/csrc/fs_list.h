// fs_list.h -- how the exclusion scorer's work list is split into runs of
// consecutive orders.  Plain C++ shared by the launches and the kernels (a
// constexpr function compiles for both sides).
#pragma once

#include <stdint.h>

namespace fs {

// The work list in n = 1 << log runs over O orders, each built by a block of
// its own: run q is orders [first(q), first(q + 1)), its entries from list +
// first(q) E.  With n <= O every run has an order, so a run's first entry lies
// in the list (the scorer's threads read it before they know whether they
// have an item); the longest run has `per` orders.
struct ListRuns {
  int log, n, O, per;
  constexpr int first(int q) const { return (int)(((int64_t)q * O) >> log); }
};

// As many runs as `most` and the orders allow, rounded down to a power of two.
constexpr ListRuns list_runs_of(int O, int64_t most) {
  int log = 0;
  while ((2 << log) <= most && (2 << log) <= O) ++log;
  return ListRuns{log, 1 << log, O, (int)((O + (1 << log) - 1) >> log)};
}

// `want` runs, or more (up to `most`) until a block can stage the longest one:
// fits(orders).  False where no run fits.
template <class F>
constexpr bool list_runs_staged(int O, int64_t want, int64_t most, F fits, ListRuns *runs) {
  for (*runs = list_runs_of(O, want); !fits(runs->per); *runs = list_runs_of(O, 2 * runs->n))
    if (2 * runs->n > most || 2 * runs->n > O) return false;
  return true;
}

}  // namespace fs
