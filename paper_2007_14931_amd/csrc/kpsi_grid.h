// Grid of the per-event kernel: plain host arithmetic, no device code.
#pragma once

#include <algorithm>
#include <cstdint>

namespace kpsi {

constexpr int64_t kPassEvents = 256;    // events of a pass: one per thread of a block
constexpr int64_t kRowPasses = 64;      // passes per block at which a call's rows are admitted
constexpr int64_t kMostPasses = 1024;   // passes per block that the kernel's product of terms holds

// Blocks of the per-event kernel over the data set and over each normalisation record: nb blocks of
// `per` passes, the first `more` of them of one more.
struct Blocks {
  int nb = 0, per = 0, more = 0;
};
struct Grid {
  Blocks d, m;
};
struct GridRule {
  int64_t cap;   // blocks resident at once
  int few;       // up to this many passes per block, no more blocks than these take
  int ept;       // passes per block set by the caller, or 0
};

inline int64_t grid_passes(int64_t n) { return (n + kPassEvents - 1) / kPassEvents; }
// Blocks of the grid at `ept` passes each.
inline int64_t blocks_at(int64_t ept, int64_t nd, int64_t nm, int nrec) {
  return (grid_passes(nd) + ept - 1) / ept + nrec * ((grid_passes(nm) + ept - 1) / ept);
}
// Rows (block partials) by which a call with a fixed row array is admitted or refused; the grids below
// take at most `limit` rows where these do.
inline int64_t grid_rows(const GridRule& r, int64_t nd, int64_t nm, int nrec) {
  return blocks_at(r.ept > 0 ? r.ept : kRowPasses, nd, nm, nrec);
}

// The grid is one resident round, or the fewest whole rounds in which no block exceeds kRowPasses
// passes.  P is the fewest passes per block at which both sets fit these slots.  Every slot is taken, P or
// fewer passes a block, the longer blocks of a set first: blocks go to the compute units in turn, so
// each unit gets as many of the longer ones as any other, to within one per set.
//   - Fewer blocks (P whole passes each, P = 2 and 3) do not shorten the longest one and leave slots idle:
//     FP64 likelihood of the large shape on 1024 slots, 1177 passes 21.2 against 19.4 us, 1638 passes 23.1
//     against 21.8 a call; FP32 gradient, 1638 passes 22.2 against 21.3.  The other way round it is at
//     most 2% (FP32, 2867 passes on 2048 slots: 21.6 against 21.9), but for the kernels with a `few`.
//   - With the longer blocks spread evenly over the set, those whose numbers differ by the count of the
//     units meet on one unit where the spread's period divides it: 1300 passes 22.8 against 20.7 us
//     (21.9 in blocks of two), 2060 passes 27.2 against 25.2.
//   - With equal whole passes per block, the 3e7 events of the largest fit run a second round that is
//     79% full: 534 against 517 us of kernel in FP32.
inline Grid pick_grid(const GridRule& r, int64_t nd, int64_t nm, int nrec, int64_t limit) {
  const int64_t td = grid_passes(nd), tm = grid_passes(nm), total = td + nrec * tm;
  Grid g;
  if (total <= 0) return g;
  auto ceil_div = [](int64_t t, int64_t p) { return (t + p - 1) / p; };
  auto equal = [&](int64_t p) {   // whole passes, the last block of a set the rest
    g.d = Blocks{(int)ceil_div(td, p), (int)p, 0};
    g.m = Blocks{(int)ceil_div(tm, p), (int)p, 0};
    return g;
  };
  auto spread = [](int64_t t, int64_t nb) { return nb > 0 ? Blocks{(int)nb, (int)(t / nb), (int)(t % nb)} : Blocks{}; };
  if (r.ept > 0) return equal(r.ept);
  int64_t rounds = ceil_div(total, kRowPasses * r.cap), slots, P;
  do {   // (a second time where the sets do not divide well: 65 passes in the fewest rounds)
    slots = std::min(limit, rounds++ * r.cap);
    P = ceil_div(total, slots);
    while (P <= kRowPasses && blocks_at(P, nd, nm, nrec) > slots) ++P;
  } while (P > kRowPasses && slots < limit);
  if (P <= r.few && slots <= r.cap) return equal(P);
  // slots in proportion to the passes, at least as many for each set as P passes per block take
  const int64_t bd = ceil_div(td, P), bm = ceil_div(tm, P);
  const int64_t nbd = std::min(td, std::max(bd, std::min((slots * td + total / 2) / total, slots - nrec * bm)));
  g.d = spread(td, nbd);
  g.m = spread(tm, std::min(tm, (slots - nbd) / nrec));
  return g;
}

// The Eq. 14 mixture: the normalisation events run in a launch of their own before the data events,
// each with a grid by its own rule.  The data set's rows are set aside before the normalisation grid is
// picked: whole rounds of it may take all that `limit` leaves.
inline Grid pick_grid_mixture(const GridRule& r, int64_t nd, int64_t nm, int nrec, int64_t limit) {
  const Grid gm = pick_grid(r, 0, nm, nrec, limit - grid_rows(r, nd, 0, 1));
  Grid g = pick_grid(r, nd, 0, 1, limit - (int64_t)nrec * gm.m.nb);
  g.m = gm.m;
  return g;
}

// Whether a grid keeps the bounds its launch relies on: rows of the partials, passes of a block.
inline bool grid_holds(const Grid& g, int nrec, int64_t limit) {
  return g.d.nb + (int64_t)nrec * g.m.nb <= limit && std::max(g.d.per + (g.d.more > 0), g.m.per + (g.m.more > 0)) <= kMostPasses;
}

}  // namespace kpsi
