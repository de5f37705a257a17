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
long rows(long cap, int ept, long nd, long nm, int nrec) { return grid_rows(GridRule{cap, false, ept}, nd, nm, nrec); }
// out: blocks of the data set and of each normalisation record, and the longest and shortest block of each
// set, from the ranges the kernel computes; returns whether the blocks cover the passes of both sets
int plan(int mix, long cap, int whole, int ept, long nd, long nm, int nrec, long limit, long* out) {
  const GridRule r{cap, whole != 0, ept};
  const Grid g = mix ? pick_grid_mixture(r, nd, nm, nrec, limit) : pick_grid(r, nd, nm, nrec, limit);
  out[0] = g.nbd;
  out[1] = g.nbm;
  bool ok = true;
  for (int s = 0; s < 2; ++s) {
    const long t = grid_passes(s ? nm : nd), nb = s ? g.nbm : g.nbd;
    const uint64_t step = s ? g.sm : g.sd;
    long most = 0, least = t, at = 0;
    for (long b = 0; b < nb; ++b) {
      const long e0 = (long)(((uint64_t)b * step) >> 32), e2 = (long)(((uint64_t)(b + 1) * step) >> 32);
      const long e1 = b + 1 < nb && e2 < t ? e2 : t;
      ok = ok && e0 == at && e1 > e0;
      at = e1;
      most = e1 - e0 > most ? e1 - e0 : most;
      least = e1 - e0 < least ? e1 - e0 : least;
    }
    ok = ok && at == t;
    out[2 + 2 * s] = most;
    out[3 + 2 * s] = least;
  }
  out[6] = grid_holds(g, nd, nm, nrec, limit);
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


def _plan(L, mix, cap, whole, ept, nd, nm, nrec, limit):
    out = (ctypes.c_long * 7)()
    covered = L.plan(mix, cap, whole, ept, nd, nm, nrec, limit, out)
    return covered, list(out)


def _sizes(seed, count):
    """Data and normalisation sizes, spread over their logarithms, the larger either one."""
    rng = random.Random(seed)
    for _ in range(count):
        nd, nm = (int(2 ** rng.uniform(0, 28.3)) for _ in range(2))
        yield rng.choice([256, 512, 768, 1024, 2048]), rng.choice([0, 1]), nd, nm, rng.choice([1, 2]), rng


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
    for cap, whole, nd, nm, nrec, rng in _sizes(17 + mix, 1500):
        ept = rng.choice([0, 0, 0, 3, 64])
        rows = shim.rows(cap, ept, nd, nm, nrec)
        for limit in (ROWS, rows, rows + 1):
            if rows > limit:
                continue
            admitted += 1
            covered, (nbd, nbm, most_d, _, most_m, _, holds) = _plan(shim, mix, cap, whole, ept, nd, nm, nrec, limit)
            assert covered and holds and nbd + nrec * nbm <= limit, (cap, whole, ept, nd, nm, nrec, limit)
            assert max(most_d, most_m) <= 1024
    assert admitted > 3000
