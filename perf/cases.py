"""Workloads by which the speed of this library is followed from change to change.

Each case is one piece of work that a program using the library repeats: a step of a fit in one
of its forms (plain, flavour-tagged, signal + background, with a moved mass), a likelihood call of
a finite-difference fit, the density of a newly loaded sample, a pseudo-experiment, and the
training and evaluation of the learned efficiency.  Models, masses and sizes are those of
`paper_2007_14931_amd.workloads` and of the studies.

Events are drawn here with torch from the case's seed: normalisation and training events flat in
phase space, data events with the K*(892) peak that dominates real data.  `exact` evaluates the
amplitude model of Eq. 2-5 and 10-12 in double precision with plain torch operations.

An FP32 context evaluates every event in single precision, so what it returns is kept as float32
here, as a single-precision optimiser keeps it; an FP64 context's results stay float64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2007_14931_amd import kpsi
from paper_2007_14931_amd import workloads as W

FLOATING = ("K*(1410)", "Z(4430)")     # lineshapes that float in the fits of the studies
PURITY, MISTAG = 0.85, 0.05            # of the signal + background and the flavour-tag studies
BATCH = 32768                          # training batch of the learned efficiency


def listed():
    return [
        # one K*(892), the smallest fit: the call's latency is what its user waits for
        dict(name="small_step_fp64", what="step", model="kstar892", precision="fp64", n_data=10_000, n_norm=100_000),
        # the benchmark's fit step: NLL and gradient of ten K* and a Z, two lineshapes floating
        dict(name="step_fp32", what="step", model="full", precision="fp32", n_data=1_000_000, n_norm=2_000_000),
        # the same step in double precision, with which such a fit is finished
        dict(name="step_fp64", what="step", model="full", precision="fp64", n_data=1_000_000, n_norm=2_000_000),
        # one likelihood call of a finite-difference gradient, on an odd number of events
        dict(name="nll_fp64", what="nll", model="full", precision="fp64", n_data=499_979, n_norm=2_000_003),
        # the largest fit: two Z, an efficiency per event, more events than the caches hold
        dict(name="large_step_fp32", what="step", model="full2z", precision="fp32", n_data=10_000_000,
             n_norm=20_000_000, efficiency=True),
        # flavour-tagged decays with a mistag fraction
        dict(name="tagged_step_fp32", what="tagged", model="full", precision="fp32", n_data=1_000_000,
             n_norm=2_000_000),
        # signal and background with efficiencies, two Z
        dict(name="mixture_step_fp32", what="mixture", model="full2z", precision="fp32", n_data=999_983,
             n_norm=2_000_000, efficiency=True),
        # two fit steps that each move a mass, with the interference matrix in use: it is rebuilt
        dict(name="moved_mass_fp32", what="moved", model="full", precision="fp32", n_data=1_000_000,
             n_norm=2_000_000),
        # a new sample is loaded and its density read back (plots, event weights)
        dict(name="density_fp64", what="density", model="full2z", precision="fp64", n_data=777_777),
        # a pseudo-experiment's data, accept-reject under the acceptance
        dict(name="toys", what="toys", model="full", precision="fp64", n_data=200_000),
        # one epoch of the learned efficiency, its last batch a partial one
        dict(name="training", what="training", n_data=1_000_000),
        # the trained network's efficiency of every normalisation event
        dict(name="network", what="network", n_data=2_000_000),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choices(["step", "nll", "tagged", "mixture", "moved", "density", "toys", "training", "network"],
                       [8, 4, 2, 2, 2, 1, 1, 1, 1])[0]
    if what in ("training", "network"):
        return dict(what=what, n_data=_log_uniform(rng, 40_000, 3_000_000))
    case = dict(what=what, model=rng.choice(["kstar892", "kstar10", "full", "full", "full2z", "full_zfree",
                                             "lass_full2z"]),
                precision=rng.choice(["fp32", "fp64"]))
    if what == "toys":
        return dict(case, precision="fp64", n_data=_log_uniform(rng, 2_000, 300_000))
    case["n_data"] = _log_uniform(rng, 3_000, 3_000_000)
    if what == "density":
        return dict(case, precision="fp64")
    case["n_norm"] = min(6_000_000, int(case["n_data"] * rng.uniform(1.5, 10.0)))
    if rng.random() < 0.5:
        case["efficiency"] = True
    return case


# ---------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _flat_masses(u):
    """m_Kpi of flat phase space (density p_B(m) q(m)) at the uniform numbers u."""
    m = torch.linspace(W.M_LO, W.M_HI, 20_001, dtype=torch.float64, device=u.device)
    k = W.KIN
    q = torch.sqrt(((m**2 - (k["mK"] + k["mPi"]) ** 2) * (m**2 - (k["mK"] - k["mPi"]) ** 2)).clamp_min(0)) / (2 * m)
    p = torch.sqrt(((k["mB"] ** 2 - (k["mJ"] + m) ** 2) * (k["mB"] ** 2 - (k["mJ"] - m) ** 2)).clamp_min(0))
    d = p * q
    c = torch.cat([torch.zeros(1, dtype=d.dtype, device=d.device), torch.cumsum(0.5 * (d[1:] + d[:-1]), 0)])
    c = c / c[-1].clone()
    i = torch.searchsorted(c, u.contiguous()).clamp(1, m.numel() - 1)
    return m[i - 1] + (m[i] - m[i - 1]) * (u - c[i - 1]) / (c[i] - c[i - 1])


def _events(n, g, peaked=False):
    """(4, n) observables on the GPU; peaked: 40% of the masses under the K*(892)."""
    u = torch.rand((4, n), dtype=torch.float64, device="cuda", generator=g)
    m = _flat_masses(u[0])
    if peaked:
        r = torch.rand((2, n), dtype=torch.float64, device="cuda", generator=g)
        peak = 0.896 + 0.03 * torch.tan(math.pi * (r[0] - 0.5))
        m = torch.where((r[1] < 0.4) & (peak > W.M_LO) & (peak < W.M_HI), peak, m)
    return torch.stack([m, 2 * u[1] - 1, 2 * u[2] - 1, math.pi * (2 * u[3] - 1)]).contiguous()


def _acceptance(ev, seed):
    """A smooth efficiency in (0.3, 0.9) over the observables."""
    co = np.random.default_rng(seed).uniform(-1.0, 1.0, 4)
    x = (2 * (ev[0] - W.M_LO) / (W.M_HI - W.M_LO) - 1, ev[1], ev[2], ev[3] / math.pi)
    return 0.3 + 0.6 * torch.sigmoid(sum(float(c) * v * (1.5 - v * v) for c, v in zip(co, x)))


def _background(ev):
    """A smooth background shape: flat in the angles but for a slope, falling in the mass."""
    return 0.2 + torch.exp(-2.0 * (ev[0] - W.M_LO)) * (1.0 + 0.5 * ev[1]) * (1.0 + 0.3 * ev[2] * torch.cos(ev[3]))


def _floating(res):
    return [r.name for r in res if r.name in FLOATING]


def _inputs(case, seed):
    """Parameters, events and per-event values of a likelihood case."""
    res = W.model(case["model"])
    g = _generator(seed)
    x = dict(res=res, params=W.params(res, seed % (1 << 31)), data=_events(case["n_data"], g, peaked=True))
    if "n_norm" in case:
        x["norm"] = _events(case["n_norm"], g)
        x["eps"] = _acceptance(x["norm"], seed) if case.get("efficiency") else None
    if case["what"] == "tagged":
        x["tags"] = torch.where(torch.rand(case["n_data"], device="cuda", generator=g) < 0.5, 1.0, -1.0).double()
    if case["what"] == "mixture":
        x["b_data"], x["b_norm"] = _background(x["data"]), _background(x["norm"])
        x["eps_data"] = _acceptance(x["data"], seed) if case.get("efficiency") else None
    if case["what"] == "moved":
        moved = x["params"].copy()
        for i, r in enumerate(res):
            if r.name in FLOATING or len(res) == 1:
                moved[W.lineshape_offset(res, i)] *= 1.001
        x["points"] = [x["params"], moved]
    return x


def _training_inputs(case, seed):
    g = _generator(seed)
    ev = _events(case["n_data"], g)
    lab = torch.rand(ev.shape[1], dtype=torch.float64, device="cuda", generator=g) < _acceptance(ev, seed)
    return ev, lab.to(torch.uint8), W.mlp_init(seed % (1 << 31))


def prepare(case, seed):
    what = case["what"]
    if what in ("training", "network"):
        ev, lab, par = _training_inputs(case, seed)
        torch.cuda.synchronize()   # the library works on a stream of its own
        e = kpsi.Engine(0, "fp64")
        e.set_model(W.KIN, W.model("kstar892"))
        return dict(what=what, engine=e, events=ev, labels=lab, params=par)
    x = _inputs(case, seed)
    res = x["res"]
    e = kpsi.Engine(0, case["precision"])
    e.set_model(W.KIN, res)
    s = dict(what=what, engine=e, params=x["params"], fp32=case["precision"] == "fp32")
    if what == "density":
        return dict(s, events=x["data"])
    if what == "toys":
        scan = _events(200_000, _generator(seed + 1))
        torch.cuda.synchronize()
        e.load(kpsi.DATA, scan)
        return dict(s, n=case["n_data"], seed=seed, smax=1.5 * float(e.density(kpsi.DATA, x["params"]).max()),
                    acceptance=W.acceptance_coefficients(seed % (1 << 31)))
    names = _floating(res)
    torch.cuda.synchronize()
    e.set_floating([1 if r.name in names else 0 for r in res])
    e.load(kpsi.DATA, x["data"])
    e.load(kpsi.NORM, x["norm"])
    if x["eps"] is not None:
        e.set_efficiency_values(x["eps"].cpu().numpy())
    if what == "tagged":
        e.set_flavour(x["tags"].cpu().numpy(), MISTAG)
    if what == "mixture":
        e.set_background(PURITY, None if x["eps_data"] is None else x["eps_data"].cpu().numpy(),
                         x["b_data"].cpu().numpy(), x["b_norm"].cpu().numpy())
    if what == "moved":
        e.set_norm_cache(1)
        s["points"] = x["points"]
    return dict(s, free=np.flatnonzero(W.free_mask(res, tuple(names))))


# ---------------------------------------------------------------- one pass
def run(state):
    e, what = state["engine"], state["what"]
    if what == "training":
        return e.mlp_train(state["params"], state["events"], state["labels"], epochs=1, batch=BATCH, lr=3e-3)
    if what == "network":
        return e.mlp_eval(state["params"], state["events"])
    if what == "density":
        e.load(kpsi.DATA, state["events"])
        return e.density(kpsi.DATA, state["params"])
    if what == "toys":
        return e.generate_model(state["params"], state["seed"], state["n"], W.PHSP_WMAX, state["smax"],
                                state["acceptance"])
    kind = np.float32 if state["fp32"] else np.float64
    if what == "nll":
        return kind(e.nll(state["params"]))
    out = []
    for p in state.get("points", [state["params"]]):
        v, g = e.nll_and_grad(p)
        out += [kind(v), g[state["free"]].astype(kind, copy=False)]
    return out


# ---------------------------------------------------------------- what a pass cannot do without
def _flops(res, grad, n_float):
    """Per event: barrier, angular and spin factors; a Breit-Wigner and complex multiply-adds per
    resonance and coupling; the adjoint of each (bench.py's operation count, by model)."""
    nc = sum(r.n_coup for r in res)
    f = 210 + 8 * len(res) + 8 * nc
    return f + (90 + 8 * nc + 45 * n_float if grad else 0)


def work(case):
    what, n = case["what"], case["n_data"]
    if what == "training":   # four observables and a label; three products of 64 x 64 and the thin layers
        return {"bytes": 33.0 * n + 2 * 4 * W.MLP_NPARAMS, "flops": 25_800.0 * n}
    if what == "network":
        return {"bytes": 40.0 * n, "flops": 8_900.0 * n}
    res = W.model(case["model"])
    if what == "density":    # four observables in, one value out; the derived kinematics once
        return {"bytes": 40.0 * n, "flops": (250.0 + _flops(res, False, 0)) * n}
    if what == "toys":       # some fifty proposals for each event that is kept
        return {"bytes": 32.0 * n, "flops": 50.0 * (450.0 + _flops(res, False, 0)) * n}
    size = 4 if case["precision"] == "fp32" else 8
    m = case["n_norm"]
    flops = _flops(res, what != "nll", len(_floating(res)))
    total = n + m
    per_data = 4.0
    if what == "tagged":
        total, per_data = 1.3 * n + 2 * m, 5.0
    if what == "mixture":
        per_data = 6.0 if case.get("efficiency") else 5.0
    w = {"bytes": size * (per_data * n + (5.0 if case.get("efficiency") else 4.0) * m), "flops": float(flops) * total}
    if what == "moved":      # two points: the data events, and the Gram product of the components
        nc = sum(r.n_coup for r in res)
        nd = 2 * sum(r.n_coup for r in res if r.name in FLOATING)
        gram = 2.0 * (2 * (2 * nc) ** 2 / 2 + 2 * (2 * nc) * (2 * nd))
        w = {"bytes": 2 * w["bytes"], "flops": 2 * (flops * n + (_flops(res, False, 0) + gram) * float(m))}
    return w


# ---------------------------------------------------------------- double precision, plain torch
def _momentum(s, a, b):
    """Breakup momentum at the squared mass s into the masses a and b."""
    x = (s - (a + b) ** 2) * (s - (a - b) ** 2)
    return torch.sqrt(x.clamp_min(0)) / (2 * torch.sqrt(s))


def _barrier(L, z):
    return [lambda z: torch.ones_like(z), lambda z: 1 + z, lambda z: 9 + 3 * z + z**2,
            lambda z: 225 + 45 * z + 6 * z**2 + z**3,
            lambda z: 11025 + 1575 * z + 135 * z**2 + 10 * z**3 + z**4][L](z)


def _small_d(J, c, s):
    """d^J_00 and d^J_10: Legendre polynomials and their derivatives."""
    p = [torch.ones_like(c), c, (3 * c**2 - 1) / 2, (5 * c**3 - 3 * c) / 2, (35 * c**4 - 30 * c**2 + 3) / 8][J]
    d = [0 * c, torch.ones_like(c), 3 * c, (15 * c**2 - 3) / 2, (35 * c**3 - 15 * c) / 2][J]
    return p, -s * d / math.sqrt(J * (J + 1)) if J else 0 * c


def _lineshape(r, M, G, s, pb_masses, q_masses):
    """Eq. 2-3, and Eq. 7-8 for the LASS S-wave: a complex amplitude for each squared mass."""
    k = W.KIN
    mB, rB, rR = k["mB"], k["rB"], k["rR"]
    LR = r.spin if r.chain == W.KSTAR else 0
    LB = (1 if r.spin == 0 else r.spin - 1) if r.chain == W.KSTAR else 1
    m = torch.sqrt(s)
    q, q0 = _momentum(s, *q_masses), _momentum(M * M, *q_masses)

    def p_of(mass):
        return torch.sqrt(((mB**2 - (pb_masses + mass) ** 2) * (mB**2 - (pb_masses - mass) ** 2)).clamp_min(0)) / (2 * mB)

    p, p0 = p_of(m), p_of(M)
    f_r = _barrier(LR, (rR * q0) ** 2) / _barrier(LR, (rR * q) ** 2)
    f_b = _barrier(LB, (rB * p0) ** 2) / _barrier(LB, (rB * p) ** 2)
    gamma = G * (q / q0) ** (2 * LR + 1) * (M / m) * f_r
    den = torch.complex(M * M - s, -M * gamma)
    front = torch.sqrt(f_b * f_r) * (p / mB) ** LB * (q / m) ** LR
    if r.shape == 1:
        u = 1 / r.lass_a + r.lass_b * q * q / 2
        e2 = torch.complex(u, q) ** 2 / (u * u + q * q)
        return front * (m * torch.complex(u, q) / (u * u + q * q) + e2 * (M * M * G / q0) / den)
    return front / den


def _z_chain(ev):
    """m^2 of J/psi pi, and Zang[l'][xi] of Eq. 10 (l' = 0, +1, -1; xi = +1, -1) from the three
    momenta in the J/psi rest frame."""
    k = W.KIN
    mB, mJ, mK, mP = k["mB"], k["mJ"], k["mK"], k["mPi"]
    m, ck, cj, phi = ev
    s = m * m
    q = _momentum(s, mK, mP)
    pb = torch.sqrt(((mB**2 - (mJ + m) ** 2) * (mB**2 - (mJ - m) ** 2)).clamp_min(0)) / (2 * mB)
    sk, sj = torch.sqrt((1 - ck**2).clamp_min(0)), torch.sqrt((1 - cj**2).clamp_min(0))
    ek, ep = torch.sqrt(mK**2 + q * q), torch.sqrt(mP**2 + q * q)
    g, gb = (mB**2 - s - mJ**2) / (2 * m * mJ), pb * mB / (m * mJ)
    o = torch.zeros_like(m)
    kaon = torch.stack([q * sk, o, g * q * ck + gb * ek], -1)
    pion = torch.stack([-q * sk, o, -g * q * ck + gb * ep], -1)
    epi = g * ep - gb * q * ck
    mz2 = mJ**2 + mP**2 + 2 * mJ * epi
    mz = torch.sqrt(mz2)
    ekz, epz = (mB**2 - mz2 - mK**2) / (2 * mz), (mz2 + mP**2 - mJ**2) / (2 * mz)
    pk, pp = torch.sqrt((ekz**2 - mK**2).clamp_min(0)), torch.sqrt((epz**2 - mP**2).clamp_min(0))
    cz = ((ekz * epz - (s - mK**2 - mP**2) / 2) / (pk * pp)).clamp(-1, 1)
    sz = torch.sqrt(1 - cz**2)
    n2 = -pion / pion.norm(dim=-1, keepdim=True)
    x2 = kaon - (kaon * n2).sum(-1, keepdim=True) * n2
    x2 = x2 / x2.norm(dim=-1, keepdim=True)
    y2 = torch.linalg.cross(n2, x2)
    n1 = torch.stack([o, o, -torch.ones_like(m)], -1)
    x1 = torch.stack([torch.ones_like(m), o, o], -1)
    y1 = torch.linalg.cross(n1, x1)
    cp, sp = torch.cos(phi)[:, None], torch.sin(phi)[:, None]
    mu = sj[:, None] * (cp * x1 + sp * y1) + cj[:, None] * n1
    ct, a, b = (mu * n2).sum(-1), (mu * x2).sum(-1), (mu * y2).sum(-1)
    st = torch.sqrt(a * a + b * b)
    cpt, spt = a / st, b / st
    xa = cj[:, None] * (cp * x1 + sp * y1) - sj[:, None] * n1
    xb = ct[:, None] * (cpt[:, None] * x2 + spt[:, None] * y2) - st[:, None] * n2
    alpha = torch.atan2((torch.linalg.cross(xb, xa) * mu).sum(-1), (xb * xa).sum(-1))
    pt = torch.atan2(spt, cpt)
    r2 = math.sqrt(0.5)
    ang = {}
    for l, dz in ((0, cz), (1, sz * r2), (-1, -sz * r2)):
        for xi in (1, -1):
            d = xi * st * r2 if l == 0 else (1 + l * xi * ct) / 2
            ang[l, xi] = dz * d * torch.polar(torch.ones_like(m), l * pt + xi * alpha)
    return mz2, ang


class _Model:
    """Per-event amplitudes a_xi as a function of the parameters (a tensor that may need gradients)."""

    def __init__(self, res, params):
        self.res, self.p = res, params
        self.ncr = sum(2 * r.n_coup for r in res)

    def density(self, ev, flips=(1.0,)):
        """S of the events read with phi -> f phi, for each f (a number, or one per event)."""
        k = W.KIN
        m, ck, cj, _ = ev
        sk, sj = torch.sqrt((1 - ck**2).clamp_min(0)), torch.sqrt((1 - cj**2).clamp_min(0))
        with_z = any(r.chain == W.ZCHAIN for r in self.res)
        mz2, ang0 = _z_chain(ev) if with_z else (None, None)
        shapes, off = [], 0
        for i, r in enumerate(self.res):
            M, G = self.p[self.ncr + 2 * i], self.p[self.ncr + 2 * i + 1]
            c = [torch.polar(self.p[off + 2 * j], self.p[off + 2 * j + 1]) for j in range(r.n_coup)]
            off += 2 * r.n_coup
            if r.chain == W.KSTAR:
                A = _lineshape(r, M, G, m * m, k["mJ"], (k["mK"], k["mPi"]))
                d0, d1 = _small_d(r.spin, ck, sk)
                c3 = [None, c[0], None] if r.spin == 0 else c
                shapes += [(A * d, l, h) for d, l, h in zip((-d1, d0, d1), (-1, 0, 1), c3) if h is not None]
            else:
                A = _lineshape(r, M, G, mz2, k["mK"], (k["mJ"], k["mPi"]))
                hs = c if len(c) == 3 else [c[0], c[1], c[1]]
                shapes += [(A, ("z", l), h) for l, h in zip((0, 1, -1), hs)]
        U = {}
        for A, l, h in shapes:
            U[l] = U.get(l, 0) + A * h
        out = []
        for f in flips:
            phi = f * ev[3]
            S = 0
            for xi in (1, -1):
                a = 0
                for l, u in U.items():
                    if isinstance(l, tuple):
                        z = ang0[l[1], xi]
                        a = a + u * torch.complex(z.real, f * z.imag)
                    else:
                        d = xi * sj * math.sqrt(0.5) if l == 0 else (1 + l * xi * cj) / 2
                        a = a + u * torch.polar(d, l * phi)
                S = S + a.real**2 + a.imag**2
            out.append(S)
        return out


def _chunks(n):
    return [(i, min(n, i + 400_000)) for i in range(0, n, 400_000)]


def _exact_step(case, x, params):
    """NLL and gradient over the free parameters, or the NLL alone."""
    res, what = x["res"], case["what"]
    grad = what != "nll"
    p = torch.tensor(params, dtype=torch.float64, device="cuda", requires_grad=grad)
    names = _floating(res)
    free = np.flatnonzero(W.free_mask(res, tuple(names)))
    nd, nm = case["n_data"], case["n_norm"]
    tagged, mixed = what == "tagged", what == "mixture"

    def summed(n, f):
        """The sums f gives over all chunks, and their gradients."""
        tot, gr = 0.0, None
        for lo, hi in _chunks(n):
            with torch.set_grad_enabled(grad):
                v = f(lo, hi)
            if grad:
                g = torch.stack([torch.autograd.grad(t, p, retain_graph=i + 1 < v.numel())[0] for i, t in enumerate(v)])
                gr = g if gr is None else gr + g
            tot = tot + v.detach()
        return tot, gr

    def norm_sums(lo, hi):
        ev = x["norm"][:, lo:hi]
        S = _Model(res, p).density(ev, (1.0, -1.0) if tagged else (1.0,))
        w = 1.0 if x["eps"] is None else x["eps"][lo:hi]
        return torch.stack([(w * s).sum() for s in S]) / nm

    I, gI = summed(nm, norm_sums)
    if tagged:
        mix = torch.tensor([[1 - MISTAG, MISTAG], [MISTAG, 1 - MISTAG]], dtype=torch.float64, device="cuda")
        N = mix @ I
        gN = mix @ gI
    else:
        N, gN = I, gI
    if mixed:
        Nb = float(x["b_norm"].double().mean())
        k = torch.tensor((1 - PURITY) / Nb, dtype=torch.float64, device="cuda")
        Np = N[0].clone().requires_grad_(grad)

    def data_sums(lo, hi):
        ev = x["data"][:, lo:hi]
        if tagged:
            q = x["tags"][lo:hi]
            S, T = _Model(res, p).density(ev, (q, -q))
            return torch.log((1 - MISTAG) * S + MISTAG * T).sum()[None]
        S = _Model(res, p).density(ev)[0]
        if mixed:
            e = 1.0 if x["eps_data"] is None else x["eps_data"][lo:hi]
            t = PURITY * e * S + k * Np * x["b_data"][lo:hi]
            if grad:   # the derivative through N, on its own
                gk.append(torch.autograd.grad(torch.log(t).sum(), Np, retain_graph=True)[0])
            return torch.log(t).sum()[None]
        return torch.log(S).sum()[None]

    gk = []
    L, gL = summed(nd, data_sums)
    if tagged:
        n = torch.stack([(x["tags"] > 0).sum(), (x["tags"] < 0).sum()]).double()
    else:
        n = torch.tensor([float(nd)], dtype=torch.float64, device="cuda")
    v = np.float64(-2 * L[0].item() + 2 * (n * torch.log(N)).sum().item())
    if not grad:
        return v
    g = -2 * gL[0] + 2 * ((n / N)[:, None] * gN).sum(0)
    if mixed:
        g = g - 2 * sum(gk) * gN[0]
    return [v, g.cpu().numpy()[free]]


def _exact_network(par, ev):
    """The network of the learned efficiency at the FP64 parameters par."""
    W1, b1, W2, b2, w3, b3 = (par[:256].view(64, 4), par[256:320], par[320:4416].view(64, 64), par[4416:4480],
                              par[4480:4544], par[4544])
    u = torch.stack([2 * (ev[0] - W.M_LO) / (W.M_HI - W.M_LO) - 1, ev[1], ev[2], ev[3] / math.pi], 1)
    h = torch.nn.functional.silu(u @ W1.T + b1)
    return torch.nn.functional.silu(h @ W2.T + b2) @ w3 + b3


def _exact_training(ev, lab, par):
    """One epoch of Adam on the mean cross-entropy."""
    p = torch.tensor(par, dtype=torch.float64, device="cuda", requires_grad=True)
    m, v, total, n = torch.zeros_like(p), torch.zeros_like(p), 0.0, ev.shape[1]
    for t, lo in enumerate(range(0, n, BATCH), 1):
        y = lab[lo:lo + BATCH].double()
        loss = torch.nn.functional.binary_cross_entropy_with_logits(_exact_network(p, ev[:, lo:lo + BATCH]), y)
        g = torch.autograd.grad(loss, p)[0]
        total += float(loss) * y.numel()
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        step = 3e-3 * (m / (1 - 0.9**t)) / (torch.sqrt(v / (1 - 0.999**t)) + 1e-8)
        p = (p.detach() - step).requires_grad_(True)
    return [p.detach().cpu().numpy(), total / n]


def exact(case, seed):
    what = case["what"]
    if what == "toys":
        return None
    if what in ("training", "network"):
        ev, lab, par = _training_inputs(case, seed)
        if what == "training":
            return _exact_training(ev, lab, par)
        p = torch.tensor(par, dtype=torch.float64, device="cuda")
        return torch.cat([torch.sigmoid(_exact_network(p, ev[:, lo:hi])) for lo, hi in _chunks(ev.shape[1])])
    x = _inputs(case, seed)
    if what == "density":
        p = torch.tensor(x["params"], dtype=torch.float64, device="cuda")
        model = _Model(x["res"], p)
        return torch.cat([model.density(x["data"][:, lo:hi])[0] for lo, hi in _chunks(case["n_data"])]).cpu().numpy()
    if what == "moved":
        return [v for p in x["points"] for v in _exact_step(case, x, p)]
    return _exact_step(case, x, x["params"])
