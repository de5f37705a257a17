// Grid of the per-event kernel: plain host arithmetic, no device code.
#pragma once

#include <algorithm>
#include <cstdint>

namespace kpsi {

constexpr int64_t kPassEvents = 256;    // events of a pass: one per thread of a block
constexpr int64_t kRowPasses = 64;      // passes per block at which a call's rows are admitted
constexpr int64_t kMostPasses = 1024;   // passes per block that the kernel's product of terms holds

// Blocks of the per-event kernel over the data set and over each normalisation record, and the passes of
// each block times 2^32 (AmpArgs::step).
struct Grid {
  int nbd = 0, nbm = 0;
  uint64_t sd = 0, sm = 0;
};
struct GridRule {
  int64_t cap;   // blocks resident at once
  bool whole;    // equal whole passes per block where one round holds them
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

// The grid is one resident round, or the fewest whole rounds that take about 64 passes per block:
// every round is full, and the passes are spread evenly over the blocks of a set, so compute units end
// together.  (With equal whole passes per block, at most 64, the 3e7 events of the largest fit ran a
// second round that was 79% full: 534 against 517 us of kernel in FP32; with flavour tags 5e6
// readings take 75.6 against 75.0 us, and 3e6 events the same 44.4 us either way.)
inline Grid pick_grid(const GridRule& r, int64_t nd, int64_t nm, int nrec, int64_t limit) {
  const int64_t td = grid_passes(nd), tm = grid_passes(nm), total = td + nrec * tm;
  Grid g;
  if (total <= 0) return g;
  auto equal = [&](int64_t ept) {
    g.nbd = (int)((td + ept - 1) / ept);
    g.nbm = (int)((tm + ept - 1) / ept);
    g.sd = g.sm = (uint64_t)ept << 32;
    return g;
  };
  if (r.ept > 0) return equal(r.ept);
  const int64_t rounds = (total + kRowPasses * r.cap - 1) / (kRowPasses * r.cap);
  const int64_t slots = std::min(limit, std::min(total, rounds * r.cap));
  if (r.whole && rounds == 1) {
    const int64_t most = std::min(r.cap, limit);
    int64_t ept = (total + most - 1) / most;
    while (ept < kRowPasses && blocks_at(ept, nd, nm, nrec) > most) ++ept;
    if (blocks_at(ept, nd, nm, nrec) <= most) return equal(ept);
  }
  // slots in proportion to the passes, at least one block where there are events
  int64_t nbd = td > 0 ? std::max<int64_t>(1, (slots * td + total / 2) / total) : 0;
  if (tm > 0) nbd = std::min(nbd, std::max<int64_t>(td > 0 ? 1 : 0, slots - nrec));
  nbd = std::min(nbd, td);
  const int64_t nbm = tm > 0 ? std::min(tm, std::max<int64_t>(1, (slots - nbd) / nrec)) : 0;
  g.nbd = (int)nbd;
  g.nbm = (int)nbm;
  g.sd = nbd > 0 ? ((uint64_t)td << 32) / (uint64_t)nbd : 0;
  g.sm = nbm > 0 ? ((uint64_t)tm << 32) / (uint64_t)nbm : 0;
  return g;
}

// The Eq. 14 mixture: the normalisation events run in a launch of their own before the data events,
// each with a grid by its own rule.  The data set's rows are set aside before the normalisation grid is
// picked: whole rounds of it may take all that `limit` leaves.
inline Grid pick_grid_mixture(const GridRule& r, int64_t nd, int64_t nm, int nrec, int64_t limit) {
  const Grid gm = pick_grid(r, 0, nm, nrec, limit - grid_rows(r, nd, 0, 1));
  Grid g = pick_grid(r, nd, 0, 1, limit - (int64_t)nrec * gm.nbm);
  g.nbm = gm.nbm;
  g.sm = gm.sm;
  return g;
}

// Whether a grid keeps the bounds its launch relies on: rows of the partials, passes of a block.
inline bool grid_holds(const Grid& g, int64_t nd, int64_t nm, int nrec, int64_t limit) {
  auto most = [](int64_t t, int64_t nb, uint64_t step) {   // passes of the longest block
    if (nb <= 0) return t;
    const int64_t last = t - (int64_t)(((uint64_t)(nb - 1) * step) >> 32);
    return std::max(last, nb > 1 ? (int64_t)((step + 0xffffffffull) >> 32) : 0);
  };
  return g.nbd + (int64_t)nrec * g.nbm <= limit && most(grid_passes(nd), g.nbd, g.sd) <= kMostPasses &&
         most(grid_passes(nm), g.nbm, g.sm) <= kMostPasses;
}

}  // namespace kpsi
