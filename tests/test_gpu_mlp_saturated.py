"""Network kernels at saturated units and huge weights: z / (1 + exp(-z)) tends to 0 for every z below -89,
also where z is of the size of the largest floats, in the evaluation and in the gradient."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2007_14931_amd import kpsi
from paper_2007_14931_amd import workloads as W
from parity_bars import check_probabilities

pytestmark = pytest.mark.gpu


def _case(seed, n=333):
    import torch
    e = kpsi.Engine(0, "fp32")
    e.set_model(W.KIN, W.model("kstar892"))
    ev = W.neutral_events(n, seed)
    lab = (np.random.default_rng(seed).uniform(size=n) < 0.5).astype(np.uint8)
    dev = torch.from_numpy(np.ascontiguousarray(ev)).to("cuda:0")
    return e, dev, torch.from_numpy(lab).to("cuda:0"), O.mlp_inputs(W.M_LO, W.M_HI, ev), lab


def _network(seed, b1, b2):
    par = W.mlp_init(seed)
    par[256:320], par[4416:4480] = b1, b2
    par[4480:4544] *= 0.01   # (the output stays away from 0 and 1)
    return par


# first-layer units from underflow of exp(-z) over the largest finite denominator (z = -88.7) to infinity
def test_gradient_with_saturated_units():
    e, dev, lab, u, y = _case(79)
    par = _network(5, np.linspace(-140.0, 140.0, 64), np.linspace(110.0, -110.0, 64))
    g, loss = e.mlp_grad(par, dev, lab)
    ref_loss, ref_p, ref_g = O.mlp(par.astype(np.float64), u, y.astype(np.float64), grad=True)
    check_probabilities(e.mlp_eval(par, dev).cpu().numpy(), ref_p, par, u)
    assert loss == pytest.approx(ref_loss, rel=2e-5)
    # the bar of the FP32 sums, and of BF16 roundings that differ in the last place (2^-8 of a unit)
    for blk in (slice(0, 256), slice(256, 320), slice(320, 4416), slice(4416, 4480), slice(4480, 4545)):
        assert np.linalg.norm(g[blk] - ref_g[blk]) <= 1e-3 * np.linalg.norm(ref_g[blk]) + 1e-9


# units far below saturation, down to the size of the largest floats: their output and slope are 0 in double
# precision, so only the unit's own zero and BF16 roundings of the others separate the results
@pytest.mark.parametrize("z", [-1e3, -1e12, -1e30, -3e38])
def test_units_far_below_zero_are_off(z):
    e, dev, lab, u, y = _case(80)
    b1, b2 = np.zeros(64), np.zeros(64)
    b1[3::7], b2[5::9] = z, z
    par = _network(6, b1, b2)
    off = par.copy()   # the same network without these units: their rows of W2 and w3 are zero
    off[320:4416].reshape(64, 64)[:, 3::7] = 0
    off[4480:4544][5::9] = 0
    p, q = e.mlp_eval(par, dev).cpu().numpy(), e.mlp_eval(off, dev).cpu().numpy()
    assert np.array_equal(p, q)
    (g, loss), (h, loss_off) = e.mlp_grad(par, dev, lab), e.mlp_grad(off, dev, lab)
    assert loss == loss_off and np.all(np.isfinite(g))
    g1, g2 = g[:256].reshape(64, 4), g[320:4416].reshape(64, 64)
    assert not g1[3::7].any() and not g[256:320][3::7].any() and not g2[:, 3::7].any()   # first layer: slope and h1
    assert not g2[5::9].any() and not g[4416:4480][5::9].any() and not g[4480:4544][5::9].any()
    keep = np.setdiff1d(np.arange(64), np.arange(3, 64, 7))
    assert np.array_equal(g[256:320][keep], h[256:320][keep])


# outputs at and beyond where 1 - p is 0 in single precision (a logit of 17), and where the loss is clamped
# at a probability of 1e-12 (27.6), for events of either label
@pytest.mark.parametrize("b3", [-60.0, -30.0, -18.0, 18.0, 30.0, 60.0])
def test_loss_of_confident_outputs(b3):
    e, dev, lab, u, y = _case(81)
    par = W.mlp_init(7)
    par[4544] = b3
    g, loss = e.mlp_grad(par, dev, lab)
    ref_loss, _, ref_g = O.mlp(par.astype(np.float64), u, y.astype(np.float64), grad=True)
    assert 0 < y.sum() < y.size and loss == pytest.approx(ref_loss, rel=2e-5)
    assert np.linalg.norm(g - ref_g) <= 1e-3 * np.linalg.norm(ref_g)
    after, train_loss = e.mlp_train(par, dev, lab, epochs=1, batch=128, lr=1e-4)
    assert np.isfinite(train_loss) and np.all(np.isfinite(after))
