"""The automatic grid of the per-event kernel against one fixed number of passes per block, where its rule
is another one (the kernels of the small shape) and for sets of very different sizes.

Per-event values are the same on both grids.  FP64: only the order of the sums differs (as in
test_gpu_grid.py).  FP32: a thread's gradient sums of up to 64 events and a wavefront's are rounded in another
order, 2^-24 each of the sum of absolute values (about 2 n); the logarithms of one product of terms per
thread carry 1e-7 each."""
import numpy as np
import pytest

from paper_2007_14931_amd import kpsi
from paper_2007_14931_amd import workloads as W

pytestmark = pytest.mark.gpu


def _compare(model, prec, nd, nm, ept):
    res = W.model(model)
    e = kpsi.Engine(0, prec)
    e.set_model(W.KIN, res)
    par = W.params(res, seed=31)
    e.load(kpsi.DATA, e.generate_phsp(43, nd, W.PHSP_WMAX))
    e.load(kpsi.NORM, e.generate_phsp(44, nm, W.PHSP_WMAX))
    auto, (auto_v, auto_g) = e.nll(par), e.nll_and_grad(par)
    e.set_events_per_thread(ept)
    ref, (ref_v, ref_g) = e.nll(par), e.nll_and_grad(par)
    f64 = prec == "fp64"
    assert max(abs(auto - ref), abs(auto_v - ref_v), abs(auto_v - auto)) <= (1e-12 if f64 else 1e-6) * 2 * nd
    ok = np.isfinite(ref_g)
    assert np.array_equal(ok, np.isfinite(auto_g))
    tol = 1e-11 if f64 else 64 * 2.0**-24
    assert np.max(np.abs(auto_g[ok] - ref_g[ok])) <= tol * max(2 * nd, np.max(np.abs(ref_g[ok])))
    e.close()


# passes of 256 events around the resident blocks (1280 and 2048), and one more event than 64 of them each
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nd,nm", [(1, 1), (300, 255), (128_001, 256_001), (262_145, 300_000), (524_289, 524_288),
                                   (4_000_001, 17_000_000), (12_000_001, 22_000_000)])
def test_small_shape(prec, nd, nm):
    _compare("kstar892", prec, nd, nm, 16)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nd,nm", [(1, 2_000_001), (700_001, 3), (21_231, 5_000_000), (3_000_000, 4_287)])
def test_sets_of_very_different_sizes(prec, nd, nm):
    _compare("full", prec, nd, nm, 3)
