"""kpsi_nll_and_grad_noalloc with the Eq. 14 mixture (two launches whose block partials share the static
array) against kpsi_nll_and_grad: bit for bit, with and without flavour tags, in both precisions, from one
event per set to more passes than resident blocks."""
import numpy as np
import pytest

from paper_2007_14931_amd import kpsi
from paper_2007_14931_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("tags", [False, True])
@pytest.mark.parametrize("nd,nm", [(1, 1), (257, 300_001), (600_011, 700_003)])
def test_noalloc_with_mixture_matches_allocating_entry_point(prec, tags, nd, nm):
    res = W.model("full")
    e = kpsi.Engine(0, prec)
    e.set_model(W.KIN, res)
    par = W.params(res, seed=61)
    e.load(kpsi.DATA, e.generate_phsp(62, nd, W.PHSP_WMAX))
    e.load(kpsi.NORM, e.generate_phsp(63, nm, W.PHSP_WMAX))
    rng = np.random.default_rng(64)
    e.set_background(0.8, rng.uniform(0.3, 0.9, nd), rng.uniform(0.1, 1.0, nd), rng.uniform(0.1, 1.0, nm))
    if tags:
        e.set_flavour(np.where(rng.random(nd) < 0.5, 1.0, -1.0), 0.1)
    v0, g0 = e.nll_and_grad(par)
    v1, g1 = e.nll_and_grad_noalloc(par)
    assert np.isfinite(v0) and v1 == v0 and np.array_equal(g1, g0, equal_nan=True)
    e.close()
