"""The grid of the per-event kernel (kpsi_grid.h) as host arithmetic: whatever the sizes, its rows stay
within the row array that the call was admitted for, every block keeps to the passes that the kernel's
product of terms holds, and the blocks cover every pass once.  Sizes run to normalisation sets of hundreds
of millions of events, which no GPU run is needed for."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "kpsi_grid.h"
using namespace kpsi;
extern "C" {
long rows(long cap, int ept, long nd, long nm, int nrec) { return grid_rows(GridRule{cap, 0, ept}, nd, nm, nrec); }
// out: blocks of the data set and of each normalisation record, and the longest and shortest block of each
// set, from the ranges the kernel computes; returns whether the blocks cover the passes of both sets
int plan(int mix, long cap, int few, int ept, long nd, long nm, int nrec, long limit, long* out) {
  const GridRule r{cap, few, ept};
  const Grid g = mix ? pick_grid_mixture(r, nd, nm, nrec, limit) : pick_grid(r, nd, nm, nrec, limit);
  out[0] = g.d.nb;
  out[1] = g.m.nb;
  bool ok = true;
  for (int s = 0; s < 2; ++s) {
    const Blocks k = s ? g.m : g.d;
    const long t = grid_passes(s ? nm : nd);
    long most = 0, least = t, at = 0;
    auto first = [&](long b) { return b * k.per + (b < k.more ? b : k.more); };
    for (long b = 0; b < k.nb; ++b) {
      const long e0 = first(b), e1 = first(b + 1) < t ? first(b + 1) : t;
      ok = ok && e0 == at && e1 > e0;
      at = e1;
      most = e1 - e0 > most ? e1 - e0 : most;
      least = e1 - e0 < least ? e1 - e0 : least;
    }
    ok = ok && at == t;
    out[2 + 2 * s] = most;
    out[3 + 2 * s] = least;
  }
  out[6] = grid_holds(g, nrec, limit);
  return ok;
}
}
"""
ROWS = 16384   # rows of the library's static array


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    src, lib = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    cxx = shutil.which("g++") or shutil.which("clang++") or "/opt/rocm/bin/amdclang++"
    subprocess.run([cxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2007_14931_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    L = ctypes.CDLL(str(lib))
    i, q = ctypes.c_int, ctypes.c_long
    L.rows.argtypes, L.rows.restype = [q, i, q, q, i], q
    L.plan.argtypes = [i, q, i, i, q, q, i, q, ctypes.POINTER(q * 7)]
    return L


def _plan(L, mix, cap, few, ept, nd, nm, nrec, limit):
    out = (ctypes.c_long * 7)()
    covered = L.plan(mix, cap, few, ept, nd, nm, nrec, limit, out)
    return covered, list(out)


def _sizes(seed, count):
    """Data and normalisation sizes, spread over their logarithms, the larger either one."""
    rng = random.Random(seed)
    for _ in range(count):
        nd, nm = (int(2 ** rng.uniform(0, 28.3)) for _ in range(2))
        yield rng.choice([256, 512, 768, 1024, 2048]), rng.choice([0, 2, 64]), nd, nm, rng.choice([1, 2]), rng


# the sizes at which whole rounds of the normalisation grid take every row (1024 and 2048 resident blocks;
# with flavour tags there are two normalisation records)
@pytest.mark.parametrize("cap,nd,nm,nrec", [
    (1024, 1_000_000, 255_000_000, 1), (1024, 1_000_000, 251_800_000, 1), (1024, 1_000_000, 126_000_000, 2),
    (2048, 1_000_000, 240_000_000, 1), (2048, 1_000_000, 117_600_000, 2), (512, 40_000_000, 220_000_000, 1)])
def test_mixture_rows_stay_within_the_static_array(shim, cap, nd, nm, nrec):
    assert shim.rows(cap, 0, nd, nm, nrec) <= ROWS   # the call is admitted
    covered, (nbd, nbm, most_d, _, most_m, _, holds) = _plan(shim, 1, cap, 0, 0, nd, nm, nrec, ROWS)
    assert covered and holds and nbd + nrec * nbm <= ROWS and max(most_d, most_m) <= 1024


@pytest.mark.parametrize("mix", [0, 1])
def test_admitted_calls_fit_their_rows(shim, mix):
    admitted = 0
    for cap, few, nd, nm, nrec, rng in _sizes(17 + mix, 1500):
        ept = rng.choice([0, 0, 0, 3, 64])
        rows = shim.rows(cap, ept, nd, nm, nrec)
        for limit in (ROWS, rows, rows + 1):
            if rows > limit:
                continue
            admitted += 1
            covered, (nbd, nbm, most_d, _, most_m, _, holds) = _plan(shim, mix, cap, few, ept, nd, nm, nrec, limit)
            assert covered and holds and nbd + nrec * nbm <= limit, (cap, few, ept, nd, nm, nrec, limit)
            assert max(most_d, most_m) <= 1024
    assert admitted > 3000


def _blocks(p, nd, nm, nrec):
    passes = lambda n: -(-n // 256)
    return -(-passes(nd) // p) + nrec * -(-passes(nm) // p)


# sets of very different sizes, and random ones: no block beyond 64 passes, and none longer than the fewest
# passes at which both sets fit the slots (a set that is small beside the other gets enough blocks)
@pytest.mark.parametrize("case", [(256, 21_231, 15_674_103, 1), (256, 20_772_885, 24_287, 1),
                                  (256, 40_000, 15_000_000, 2), (1024, 1, 200_000_000, 1), "random"])
def test_no_block_is_longer_than_it_has_to_be(shim, case):
    if case == "random":
        cases = [(cap, nd, nm, nrec) for cap, _, nd, nm, nrec, _ in _sizes(5, 1500)]
    else:
        cases = [case]
    for cap, nd, nm, nrec in cases:
        for few in (0, 2, 64):
            covered, (nbd, nbm, most_d, least_d, most_m, least_m, _) = _plan(shim, 0, cap, few, 0, nd, nm, nrec, 1 << 40)
            used = nbd + nrec * nbm
            most = max(most_d, most_m)
            rounds = -(-used // cap)
            assert covered and most <= 64, (cap, nd, nm, nrec, few)
            assert most == 1 or _blocks(most - 1, nd, nm, nrec) > rounds * cap
            # whole rounds are full, but for the passes that run out and the records' common block count
            if few == 0:
                assert used > rounds * cap - nrec or most == 1
                assert most_d - least_d <= 1 and most_m - least_m <= 1


# at few passes per block a kernel with `few` takes no more blocks than these need
@pytest.mark.parametrize("nd,nm", [(2060 * 85, 2060 * 171), (1500 * 85, 1500 * 171), (100, 256 * 1400)])
def test_few_passes_take_the_fewest_blocks(shim, nd, nm):
    _, (nbd, nbm, most_d, _, most_m, _, _) = _plan(shim, 0, 1280, 2, 0, nd, nm, 1, 1 << 40)
    assert max(most_d, most_m) == 2 and nbd + nbm == _blocks(2, nd, nm, 1)
