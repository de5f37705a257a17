"""The automatic grid of the per-event kernel covers every event once, at the sizes where its rule
changes: fewer passes (of 256 events) than resident blocks, one more, a fraction of a pass per block,
and one more event than one round of 64 passes per block holds.

The reference is the same likelihood on a grid of one fixed number of passes per block
(`set_events_per_thread`).  Only the order of the FP64 sums differs: n terms summed in blocks, each
rounding at most 2^-53 of a partial sum, and the NLL is the difference of two such sums of about
n (mean |ln S|) each; 1e-12 of 2 n is 9000 roundings of the total.
"""
import numpy as np
import pytest

from paper_2007_14931_amd import kpsi
from paper_2007_14931_amd import workloads as W

pytestmark = pytest.mark.gpu


def _engine(model, prec, nd, nm):
    res = W.model(model)
    e = kpsi.Engine(0, prec)
    e.set_model(W.KIN, res)
    par = W.params(res, seed=31)
    e.load(kpsi.DATA, e.generate_phsp(41, nd, W.PHSP_WMAX))
    e.load(kpsi.NORM, e.generate_phsp(42, nm, W.PHSP_WMAX))
    return e, par


# cap: resident blocks (256 compute units x 2..8 per unit); 256 x 1024 and 256 x 2048 events are one
# pass per block of the gradient and the likelihood-only kernels, 16.8e6 is 64 passes of 1024 blocks
@pytest.mark.parametrize("nd,nm", [(1, 1), (257, 1), (100_000, 162_144), (100_001, 162_144),
                                   (262_145, 262_144), (300_007, 700_013), (3_000_001, 13_777_217)])
def test_automatic_grid_covers_every_event(nd, nm):
    e, par = _engine("full", "fp64", nd, nm)
    auto, (auto_v, auto_g) = e.nll(par), e.nll_and_grad(par)
    e.set_events_per_thread(16)
    ref, (ref_v, ref_g) = e.nll(par), e.nll_and_grad(par)
    tol = 1e-12 * 2 * nd
    assert abs(auto - ref) <= tol and abs(auto_v - ref_v) <= tol and abs(auto_v - auto) <= tol
    ok = np.isfinite(ref_g)
    assert np.array_equal(ok, np.isfinite(auto_g))
    assert np.max(np.abs(auto_g[ok] - ref_g[ok])) <= 1e-11 * max(2 * nd, np.max(np.abs(ref_g[ok])))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_automatic_grid_with_flavour_tags_and_mixture(prec):
    nd, nm = 70_001, 130_003
    e, par = _engine("full", prec, nd, nm)
    rng = np.random.default_rng(5)
    e.set_background(0.8, rng.uniform(0.3, 0.9, nd), rng.uniform(0.1, 1.0, nd), rng.uniform(0.1, 1.0, nm))
    e.set_flavour(np.where(rng.random(nd) < 0.5, 1.0, -1.0), 0.1)
    v, g = e.nll_and_grad(par)
    e.set_events_per_thread(3)
    w, h = e.nll_and_grad(par)
    # FP32: per-event values are the same; FP32 sums of up to three events per thread and then of 64
    # lanes are rounded in another order (2^-24 each of the sum of absolute values, about 2 nd)
    tol = (1e-12 if prec == "fp64" else 3e-6) * 2 * nd
    ok = np.isfinite(h)
    assert abs(v - w) <= 1e-12 * 2 * nd if prec == "fp64" else abs(v - w) <= 1e-7 * 2 * nd
    assert np.array_equal(ok, np.isfinite(g)) and np.max(np.abs(g[ok] - h[ok])) <= tol
