"""The constant factors of the lambda = +-1 terms beside those of lambda = 0, in double precision.

For a K* of spin 1 alone, S of H = (0, 0, 1) over S of H = (0, 1, 0) is
(1 - cos^2 theta_K)(1 + cos^2 theta_J) / (4 cos^2 theta_K (1 - cos^2 theta_J)): the lineshape cancels, and the
factor between the two terms, -1/2, is a number without rounding.  The mean relative error over n events is that of
the factors: each event's roundings (a few 2^-53) average out to below 1e-17 for 2e5 events.  A factor put
together from two rounded 1/sqrt2 is off by 2^-52, which shifts S by 4e-16."""
import numpy as np
import pytest

from paper_2007_14931_amd import kpsi
from paper_2007_14931_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["K*(892)", "K*(1410)", "K*(1680)"])
def test_helicity_terms_have_exact_relative_scale(name):
    res = [r for r in W.KSTARS if r.name == name]
    e = kpsi.Engine(0, "fp64")
    e.set_model(W.KIN, res)
    ev = e.generate_phsp(91, 200_000, W.PHSP_WMAX)
    e.load(kpsi.DATA, ev)
    S = []
    for h in ((0, 0, 1), (0, 1, 0)):
        par = W.params(res, seed=1)
        par[0:6:2], par[1:6:2] = h, 0.0
        S.append(e.density(kpsi.DATA, par).astype(np.longdouble))
    ck, cj = (ev[i].cpu().numpy().astype(np.longdouble) for i in (1, 2))
    want = (1 - ck**2) * (1 + cj**2) / (4 * ck**2 * (1 - cj**2))
    d = S[0] / S[1] / want - 1
    print(f"[parity] {name}: mean {float(d.mean()):.2e} rms {float(np.sqrt(np.mean(d**2))):.2e}", flush=True)
    assert abs(d.mean()) <= 1e-16
    e.close()
