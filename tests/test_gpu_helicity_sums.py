"""Gradient of a small helicity coupling beside a large one, in single precision.

The terms of a lambda = -1 gradient average out over phase space when H_-1 is small (helicities are
orthogonal), so its FP32 sums stay far below those of lambda = +1 and must not carry their rounding.  The same
likelihood with 1024 events per thread and with one (where the thread sums do not round) differs only by the
rounding of these sums.  Emulated in numpy for one K*(892) with |H_-1| = 1e-3 and 2^20 events: per event 1e-9
(at most 2.7e-9) summed by helicity, 4e-9 to 5e-8 (4e-8 rms) as the difference of two sums of the large
helicity's size.  The bar is 1e-8 for the rms over the small couplings and three samples."""
import dataclasses

import numpy as np
import pytest

from paper_2007_14931_amd import kpsi
from paper_2007_14931_amd import workloads as W

pytestmark = pytest.mark.gpu
N = 1 << 20


@pytest.mark.parametrize("model", ["kstar892", "kstar10", "z_free"])
def test_small_helicity_beside_a_large_one(model):
    res = W.model(model) if model != "z_free" else [dataclasses.replace(W.Z4430, hel_free=True)]
    par = W.params(res, seed=3)
    small = []
    for i, r in enumerate(res):
        k = W.coupling_offset(res, i)
        if r.chain == W.KSTAR and r.spin == 0:
            continue
        small.append(k + (0 if r.chain == W.KSTAR else 4))   # lambda = -1 of (-1, 0, +1), lambda' = -1 of (0, +1, -1)
        par[k:k + 6:2] = 1.0
        par[small[-1]] = 1e-3
    e = kpsi.Engine(0, "fp32")
    e.set_model(W.KIN, res)
    d = []
    for seed in (71, 72, 73):
        e.load(kpsi.DATA, e.generate_phsp(seed, N, W.PHSP_WMAX))
        e.load(kpsi.NORM, e.generate_phsp(seed + 10, N, W.PHSP_WMAX))
        g = []
        for ept in (1024, 1):
            e.set_events_per_thread(ept)
            g.append(e.nll_and_grad(par)[1][small])
        d.append((g[0] - g[1]) / N)
    rms = float(np.sqrt(np.mean(np.square(d))))
    print(f"[parity] {model}: rms {rms:.2e} per event", flush=True)
    assert rms <= 1e-8
    e.close()


def _gradients(prec, res, par, seed, n, cache):
    e = kpsi.Engine(0, prec)
    e.set_model(W.KIN, res)
    e.load(kpsi.DATA, e.generate_phsp(seed, n, W.PHSP_WMAX))
    e.load(kpsi.NORM, e.generate_phsp(seed + 10, n, W.PHSP_WMAX))
    e.set_norm_cache(cache)
    g = e.nll_and_grad(par)[1]
    e.close()
    return g


# The coupling constants themselves: the gradient of H_-1 is 2 n I_{--} H_-1 / S (a third of 4 n per unit of H here),
# so an H_-1 known only to the rounding of a large H_+1 (2^-25, as half the difference of two rounded sums)
# moves it by about 1e-8 per event, in every event alike, while the roundings of single events average out:
# 3e-9 for 2^20 events, 1.5e-9 for 2^22.
def test_small_coupling_constants_beside_large_ones():
    res = W.model("kstar892")
    rng = np.random.default_rng(8)
    d = []
    for seed in range(6):
        par = W.params(res, seed=3)
        par[0:6:2] = 1e-3, rng.uniform(0.5, 1.5), rng.uniform(0.5, 1.5)
        g = [_gradients(p, res, par, 171 + seed, 4 * N, 0)[0] for p in ("fp32", "fp64")]
        d.append((g[0] - g[1]) / (4 * N))
    rms = float(np.sqrt(np.mean(np.square(d))))
    print(f"[parity] coupling constants: rms {rms:.2e} per event", flush=True)
    assert rms <= 4e-9
