"""Performance cases: the calls that programs built on this library make, over
the range of sizes that they meet, with a plain 64-bit reference for each.

A case is a dict of plain values:

  form      "toa" (per-TOA form) or "std" (standardized form)
  call      "eval" (log p and gradient), "autograd" (LogPosterior forward and
            backward), "hmc" (one trajectory of `leapfrog` steps, graph replay)
            or "coef" (evaluation and the coefficients of the same points)
  n_psr, n_toa, nf_rn, nf_gw, nf_dm, chains     sizes (n_toa over all pulsars)
  cw        a continuous wave is sampled too (`cw_nf` harmonics in the
            standardized form's own basis)
  free, tm, tempered, split    standardized form: free spectra, columns of a
            stored design matrix (0: offset and quadratic), a temperature
            ladder, split common-process / pulsar-noise coefficients
  tiles, waves, place          tuning of the TOA pass; tiles 0 takes the chunk
            length that fits the data set (with one wave a workgroup as a
            server does), tiles -1 leaves the data set's default

Data are drawn from the seed: pulsars uniform on the sky, ragged TOA counts,
uncertainties of 10^-6 s within a decade or so, one to four backends per
pulsar, residuals of white noise plus a random walk of 1 us.
"""
import math

import numpy as np
import torch

from paper_2607_06834_amd import api, autotune

YEAR = 365.25 * 86400.0
LN10 = math.log(10.0)
LN2PI = math.log(2.0 * math.pi)
SEED = 203                       # of the momenta and accept draws

DEFAULTS = dict(nf_rn=10, nf_gw=10, nf_dm=0, cw=False, cw_nf=0, free=False, tm=0, tempered=False,
                split=False, leapfrog=0, tiles=-1, waves=1, place=1)


def _case(**kw):
    return {**DEFAULTS, **kw}


def listed():
    return [
        # One point of a three-pulsar array through the raw call: the smallest
        # call there is, as an optimiser or a diagnostic makes it in a loop.
        _case(name="toa_eval_3psr_1chain", form="toa", call="eval", n_psr=3, n_toa=1500, chains=1),
        # The same kind of array with a continuous wave through torch's
        # autograd, forward and backward, at an odd number of chains: a
        # variational fit or a custom sampler written in torch.
        _case(name="toa_autograd_cw_3psr_33chains", form="toa", call="autograd", n_psr=3, n_toa=1500, chains=33,
              cw=True),
        # A whole trajectory of many chains on a small array.
        _case(name="toa_hmc_3psr_256chains", form="toa", call="hmc", n_psr=3, n_toa=1500, chains=256, leapfrog=20),
        # One evaluation of the benchmark's array (67 pulsars, 250k TOAs, 64
        # chains), with workgroups of four waves that fill one round of the
        # device: what the autotuner finds there.
        _case(name="toa_eval_67psr_64chains", form="toa", call="eval", n_psr=67, n_toa=250_000, nf_rn=30, nf_gw=14,
              nf_dm=30, chains=64, tiles=0, waves=4, place=2),
        # A whole trajectory of it: the benchmark's own step.
        _case(name="toa_hmc_67psr_64chains", form="toa", call="hmc", n_psr=67, n_toa=250_000, nf_rn=30, nf_gw=14,
              nf_dm=30, chains=64, leapfrog=20, tiles=0, waves=4, place=2),
        # A served request with a continuous wave, 16 chains as the server runs it.
        _case(name="toa_eval_cw_45psr_16chains", form="toa", call="eval", n_psr=45, n_toa=60_001, nf_rn=17, nf_gw=17,
              nf_dm=17, cw=True, chains=16, tiles=0),
        # The largest array that the server's stream of requests holds.
        _case(name="toa_hmc_120psr_16chains", form="toa", call="hmc", n_psr=120, n_toa=140_003, nf_rn=30, nf_gw=30,
              nf_dm=30, chains=16, leapfrog=5, tiles=0),
        # The paper's own evaluation at the benchmark's array: Gram form, 120
        # coefficients a pulsar.
        _case(name="std_eval_67psr_64chains", form="std", call="eval", n_psr=67, n_toa=67_000, nf_rn=30, nf_gw=14,
              nf_dm=30, chains=64),
        # The paper's simulated array of 100 pulsars with a continuous wave in
        # its own basis of 60 frequencies.
        _case(name="std_eval_cw_100psr_64chains", form="std", call="eval", n_psr=100, n_toa=18_000, nf_rn=30,
              nf_gw=14, cw=True, cw_nf=60, chains=64),
        # Separate coefficients of the common process and of the pulsars.
        _case(name="std_eval_split_67psr_64chains", form="std", call="eval", n_psr=67, n_toa=67_000, nf_rn=30,
              nf_gw=14, nf_dm=30, chains=64, split=True),
        # A ragged array with a stored design matrix and free spectra along a
        # temperature ladder, points and their coefficients: what a
        # tempered sampler's bookkeeping asks for.
        _case(name="std_coef_free_33psr_17chains", form="std", call="coef", n_psr=33, n_toa=9_001, nf_rn=13,
              nf_gw=9, nf_dm=5, chains=17, free=True, tm=8, tempered=True),
        # A trajectory of a small run in the paper's form: a few chains, where
        # each evaluation is a handful of short launches.
        _case(name="std_hmc_20psr_8chains", form="std", call="hmc", n_psr=20, n_toa=5_000, nf_rn=20, nf_gw=10,
              nf_dm=0, chains=8, leapfrog=10),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        form = rng.choice(["toa", "std"])
        n_psr = _log_int(rng, 2, 120)
        nf_rn, nf_gw = rng.randint(3, 30), rng.randint(3, 30)
        c = _case(form=form, n_psr=n_psr, nf_rn=nf_rn, nf_gw=nf_gw, nf_dm=rng.choice([0, rng.randint(3, 30)]),
                  chains=_log_int(rng, 1, 256), cw=rng.random() < 0.3)
        if form == "toa":
            c["call"] = rng.choice(["eval", "autograd", "hmc"])
            c["n_toa"] = n_psr * _log_int(rng, 200, 4000) + rng.randint(0, 15)
            c["tiles"] = rng.choice([0, 0, -1])
        else:
            c["call"] = rng.choice(["eval", "coef", "hmc"])
            c["n_toa"] = n_psr * _log_int(rng, 100, 1000) + rng.randint(0, 15)
            c["free"], c["tempered"] = rng.random() < 0.3, rng.random() < 0.3
            c["tm"] = rng.choice([0, 0, rng.randint(4, 12)])
            c["split"] = rng.random() < 0.25
            c["cw_nf"] = rng.randint(20, 60) if c["cw"] else 0
        if c["call"] == "hmc":
            c["leapfrog"] = rng.randint(2, 20)
        # Within the largest listed case of its form, and with the dense
        # priors of many pulsars within theirs.
        dense = c["chains"] * c["nf_gw"] * max(1, c["leapfrog"]) * n_psr ** 3
        top = max((x for x in listed() if x["form"] == form), key=lambda x: work(x)["flops"])
        if work(c)["flops"] <= work(top)["flops"] and dense <= 16 * 30 * 5 * 120 ** 3:
            return c


# ------------------------------------------------------------------- inputs --

def _array(case, seed):
    """A data set's description, as api.Dataset and api.StdDataset take it."""
    r = np.random.default_rng([seed, case["n_psr"], case["n_toa"]])
    n, total = case["n_psr"], case["n_toa"]
    ka = max(case["nf_rn"], case["nf_gw"])
    span = (10.0 if n < 10 else 15.0 if case["form"] == "std" else 16.0) * YEAR
    cth, phi = r.uniform(-1.0, 1.0, n), r.uniform(0.0, 2.0 * np.pi, n)
    sth = np.sqrt(1.0 - cth * cth)
    raw = 10.0 ** r.normal(0.0, 0.2, n)
    low = min(total // n, 2 * (ka + case["nf_dm"]) + case["tm"] + 10)
    counts = low + np.floor(raw / raw.sum() * (total - low * n)).astype(np.int64)
    counts[0] += total - counts.sum()
    off = np.concatenate([[0], np.cumsum(counts)])
    backends = r.integers(1, 5, n)
    first = np.concatenate([[0], np.cumsum(backends)])
    t, backend = np.empty(total), np.empty(total, np.int32)
    for i in range(n):
        t[off[i]:off[i + 1]] = np.sort(r.uniform(0.0, span, counts[i]))
        backend[off[i]:off[i + 1]] = first[i] + r.integers(0, backends[i], counts[i])
    sigma = 10.0 ** (-6.0 + 0.7 * np.clip(r.standard_normal(total), -3.0, 3.0))
    dt = 1.1 * sigma * r.standard_normal(total)
    for i in range(n):
        s = slice(off[i], off[i + 1])
        walk = np.cumsum(np.sqrt(np.diff(t[s], prepend=0.0) / span) * r.standard_normal(counts[i]))
        dt[s] += 1e-6 * (walk - walk.mean())
    d = dict(n_psr=n, toa_offsets=off, t=t, dt=dt, sigma=sigma, nu=r.uniform(0.4e9, 2.0e9, total), backend=backend,
             efac=np.full(first[-1], 1.1), equad=np.full(first[-1], 10.0 ** -6.5),
             psr_pos=np.stack([sth * np.cos(phi), sth * np.sin(phi), cth], axis=1), tspan=span,
             nf_rn=case["nf_rn"], nf_gw=case["nf_gw"], nf_dm=case["nf_dm"], dm_scale=1.4e9 ** 2, sigma_b=1e-5,
             has_cw=int(case["cw"]))
    if case["form"] == "std":
        d.update(spectrum="free" if case["free"] else "powerlaw", split=int(case["split"]))
        if case["cw"]:
            d.update(cw_nf=case["cw_nf"], cw_tspan=2.0 * span)
        if case["tm"]:
            yr, u = 2.0 * np.pi * t / YEAR, t / span
            cols = [np.ones(total), u, u * u, np.sin(yr), np.cos(yr)] + [r.standard_normal(total) for _ in range(7)]
            d["tm"] = np.stack(cols[:case["tm"]], axis=1)
    if case["free"]:
        m = case["nf_gw"] + n * (case["nf_rn"] + case["nf_dm"])
        lo, hi = np.full(m, -20.0), np.full(m, -5.0)
    else:
        m = (case["nf_gw"] > 0) + n * ((case["nf_rn"] > 0) + (case["nf_dm"] > 0))
        lo, hi = np.tile([-20.0, 0.0], m), np.tile([-10.0, 7.0], m)
    if case["cw"]:
        lo = np.concatenate([lo, [-1.0, 0.0, 7.0, -9.0, 0.0, -1.0, 0.0, -18.0]])
        hi = np.concatenate([hi, [1.0, 2 * np.pi, 10.0, -7.5, 2 * np.pi, 1.0, np.pi, -11.0]])
    d.update(prior_lo=lo, prior_hi=hi)
    return d


def _widths(case):
    """Entries of theta (without the CW's), of u and of the coefficients of a point."""
    n, ka = case["n_psr"], max(case["nf_rn"], case["nf_gw"])
    th = case["nf_gw"] + n * (case["nf_rn"] + case["nf_dm"]) if case["free"] else \
        2 * ((case["nf_gw"] > 0) + n * ((case["nf_rn"] > 0) + (case["nf_dm"] > 0)))
    if case["split"]:
        z = 2 * (case["nf_gw"] + case["nf_rn"] + case["nf_dm"])
    else:
        z = 2 * (ka + case["nf_dm"])
    return th, 3 * n if case["form"] == "toa" else 0, n * z


def _points(case, seed):
    """Points around one set of hyper-parameters, as a sampler's chains are, and beta."""
    r = np.random.default_rng([seed, 1, case["chains"]])
    th, u, z = _widths(case)
    C, n = case["chains"], case["n_psr"]
    if case["free"]:
        mid = r.uniform(-15.5, -12.5, th)
    else:
        mid = np.empty(th)
        mid[0::2], mid[1::2] = r.uniform(-16.0, -13.0, th // 2), r.uniform(2.0, 5.0, th // 2)
        mid[:2] = -14.5, 13.0 / 3.0
    x = mid + r.uniform(-0.05, 0.05, (C, th))
    parts = [x]
    if case["cw"]:
        cw = np.array([r.uniform(-0.7, 0.7), r.uniform(0.5, 5.5), r.uniform(8.3, 8.9), r.uniform(-8.4, -8.0),
                       r.uniform(0.5, 5.5), r.uniform(-0.7, 0.7), r.uniform(0.5, 2.5), r.uniform(-14.8, -13.8)])
        parts.append(cw + r.uniform(-0.02, 0.02, (C, 8)))
    parts.append(r.standard_normal((C, u + z)))
    beta = 0.6 ** np.linspace(0.0, 6.0, C) if case["tempered"] else None
    return np.concatenate(parts, axis=1), beta


def _inv_mass(case, d):
    """Hyper-parameters move slowly beside the whitened coefficients."""
    im = np.ones(d)
    im[: _widths(case)[0] + 8 * case["cw"]] = 1e-8 if case["form"] == "toa" else 1e-4
    return im


def _eps(case):
    return 1e-4 if case["form"] == "toa" else 0.02


# --------------------------------------------------------------------- call --

def prepare(case, seed):
    d = _array(case, seed)
    x, beta = _points(case, seed)
    g = api.Dataset(d) if case["form"] == "toa" else api.StdDataset(d)
    s = dict(case=case, g=g, x=torch.tensor(x, device="cuda"),
             beta=None if beta is None else torch.tensor(beta, device="cuda"))
    if case["form"] == "toa" and case["tiles"] >= 0:
        cu = torch.cuda.get_device_properties(0).multi_processor_count
        if case["tiles"]:
            tuning = case["tiles"], case["waves"], case["place"]
        elif case["waves"] == 1:
            tuning = autotune.serving_tuning(d["toa_offsets"], case["chains"], cu)
        else:
            fit = autotune.round_fitting_tpcs(d["toa_offsets"], case["chains"], cu, wpb=case["waves"], rounds=(1,),
                                              waves_per_simd=(2,))
            tuning = fit[0], case["waves"], case["place"]
        g.ptafs_set_tuning(*tuning)
    if case["call"] == "autograd":
        s["x"].requires_grad_(True)
    if case["call"] == "hmc":
        s["logp"], s["grad"], _ = _evaluate(s)
        s["accept"] = torch.zeros(case["chains"], dtype=torch.int64, device="cuda")
        s["inv_mass"] = torch.tensor(_inv_mass(case, x.shape[1]), device="cuda")
        s["traj"] = 0
    return s


def _evaluate(s):
    if s["case"]["form"] == "toa":
        return s["g"].ptafs_logp_grad(s["x"])
    return s["g"].ptafs_std_logp_grad(s["x"], beta=s["beta"])


def run(state):
    s, case, g = state, state["case"], state["g"]
    if case["call"] == "hmc":
        kw = dict(n_traj=1, n_leapfrog=case["leapfrog"], eps=_eps(case), seed=SEED, traj0=s["traj"],
                  inv_mass=s["inv_mass"])
        if case["form"] == "toa":
            g.ptafs_hmc_run(s["x"], s["logp"], s["grad"], s["accept"], **kw)
        else:
            g.ptafs_std_hmc_run(s["x"], s["logp"], s["grad"], s["accept"], beta=s["beta"], **kw)
        s["traj"] += 1
        return dict(x=s["x"], logp=s["logp"], grad=s["grad"], accept=s["accept"])
    if case["call"] == "autograd":
        s["x"].grad = None
        logp, status = api.LogPosterior.apply(s["x"], g)
        logp.sum().backward()
        return dict(logp=logp.detach(), grad=s["x"].grad, status=status)
    logp, grad, status = _evaluate(s)
    out = dict(logp=logp, grad=grad, status=status)
    if case["call"] == "coef":
        out["coef"] = g.ptafs_std_coefficients(s["x"], beta=s["beta"])
    return out


def work(case):
    n, C, N = case["n_psr"], case["chains"], case["n_toa"]
    ka, kd, kg = max(case["nf_rn"], case["nf_gw"]), case["nf_dm"], case["nf_gw"]
    th, u, z = _widths(case)
    d = th + 8 * case["cw"] + u + z
    prior = C * kg * float(n) ** 3                      # factor, inverse and its product with chol(Gamma)
    io = 8.0 * C * (2 * d + 1)
    if case["form"] == "toa":
        toa = N * C * (8.0 * (ka + kd) + 19.0 + 80.0 * case["cw"])
        one = dict(bytes=32.0 * N + io, flops=toa + prior + 20.0 * C * kg * n * n)
    else:
        sets = [2 * (ka + kd)] + ([2 * kg, 2 * (case["nf_rn"] + kd)] if case["split"] else [])
        fac = sum(2.0 * P ** 3 / 3.0 + 12.0 * P * P for P in sets) * n * C
        k2 = 2 * case["cw_nf"]
        cw = C * n * 4.0 * k2 * (2 * k2 + sets[0])
        one = dict(bytes=8.0 * n * (sets[0] ** 2 / 2 + k2 * (k2 / 2 + sets[0])) + io,
                   flops=fac + cw + (0.0 if case["split"] else prior))
    if case["call"] == "hmc":
        one = dict(bytes=one["bytes"] * case["leapfrog"] + 32.0 * C * d, flops=one["flops"] * case["leapfrog"])
    elif case["call"] == "coef":
        one["bytes"] += 8.0 * C * z
        one["flops"] += fac
    return one


# ---------------------------------------------------------------- reference --

def _hd(pos):
    b = 0.5 * (1.0 - np.clip(pos @ pos.T, -1.0, 1.0))
    np.fill_diagonal(b, 1.0)
    g = 1.5 * b * np.log(b) - 0.25 * b + 0.5
    np.fill_diagonal(g, 1.0)
    return torch.tensor(g)


def _cw_delay(p, t, pos):
    """Earth-term delay of a circular binary, p (C, 8) at times t for one pulsar: (C, len(t))."""
    cth, phi, lmc, lf, phi0, ci, psi, lh = (p[:, j:j + 1] for j in range(8))
    m, w0 = 10.0 ** lmc * 4.925490947641e-6, math.pi * 10.0 ** lf
    y = 256.0 / 5.0 * m ** (5.0 / 3.0) * w0 ** (8.0 / 3.0) * t
    l1 = torch.log1p(-y)
    w = w0 * torch.exp(-0.375 * l1)
    ph = phi0 - torch.expm1(0.625 * l1) / (32.0 * (m * w0) ** (5.0 / 3.0))
    sth = torch.sqrt(1.0 - cth * cth)
    mp = torch.sin(phi) * pos[0] - torch.cos(phi) * pos[1]
    nq = -cth * torch.cos(phi) * pos[0] - cth * torch.sin(phi) * pos[1] + sth * pos[2]
    om = -(sth * torch.cos(phi) * pos[0] + sth * torch.sin(phi) * pos[1] + cth * pos[2])
    fp, fx = 0.5 * (mp * mp - nq * nq) / (1.0 + om), mp * nq / (1.0 + om)
    alpha = 10.0 ** lh / (2.0 * w0 ** (2.0 / 3.0) * w ** (1.0 / 3.0))
    P, Q = -torch.sin(2.0 * ph) * (1.0 + ci * ci), 2.0 * torch.cos(2.0 * ph) * ci
    c2, s2 = torch.cos(2.0 * psi), torch.sin(2.0 * psi)
    return -alpha * (P * (fp * c2 + fx * s2) + Q * (fx * c2 - fp * s2))


class _Reference:
    """log p and its gradient by autograd of the plain definition, on the CPU."""

    def __init__(self, case, d):
        self.case, self.d = case, d
        self.ka, self.kd = max(case["nf_rn"], case["nf_gw"]), case["nf_dm"]
        self.gamma = _hd(d["psr_pos"])
        f = torch.arange(1, max(self.ka, self.kd) + 1, dtype=torch.float64) / d["tspan"]
        self.lnfy = torch.log(f * YEAR)
        self.box = float(np.sum(np.log(d["prior_hi"] - d["prior_lo"])))
        self.psr = [self._pulsar(i) for i in range(case["n_psr"])]

    def _pulsar(self, i):
        case, d = self.case, self.d
        s = slice(int(d["toa_offsets"][i]), int(d["toa_offsets"][i + 1]))
        t, dt = d["t"][s], d["dt"][s]
        k = np.arange(1, max(self.ka, self.kd) + 1)
        arg = 2.0 * np.pi * np.outer(t, k) / d["tspan"]
        F = np.stack([np.sin(arg), np.cos(arg)], axis=2).reshape(t.size, -1)
        w = d["dm_scale"] / d["nu"][s] ** 2
        T = np.concatenate([F[:, :2 * self.ka], w[:, None] * F[:, :2 * self.kd]], axis=1)
        b = d["backend"][s]
        N = (d["efac"][b] * d["sigma"][s]) ** 2 + d["equad"][b] ** 2
        tau = (t - 0.5 * (t.min() + t.max())) / (0.5 * (t.max() - t.min()))
        M = np.stack([np.ones_like(tau), tau, tau * tau], axis=1)
        if case["form"] == "toa":
            return dict(t=torch.tensor(t), dt=torch.tensor(dt), T=torch.tensor(T), M=torch.tensor(M),
                        N=torch.tensor(N))
        if case["tm"]:
            M = d["tm"][s]
        Mw, Tw, dw = M / np.sqrt(N)[:, None], T / np.sqrt(N)[:, None], dt / np.sqrt(N)
        q, rr = np.linalg.qr(Mw)
        Tw, dw = Tw - q @ (q.T @ Tw), dw - q @ (q.T @ dw)
        ld = np.sum(np.log(N)) + 2.0 * np.sum(np.log(np.abs(np.diag(rr)))) - np.linalg.slogdet(M.T @ M)[1]
        out = dict(S0=Tw.T @ Tw, d=Tw.T @ dw, c=float(dw @ dw),
                   k=-0.5 * ((t.size - M.shape[1]) * LN2PI + ld))
        if case["cw"]:
            arg = 2.0 * np.pi * np.outer(t, np.arange(1, case["cw_nf"] + 1)) / d["cw_tspan"]
            FD = np.stack([np.sin(arg), np.cos(arg)], axis=2).reshape(t.size, -1) / np.sqrt(N)[:, None]
            FD = FD - q @ (q.T @ FD)
            out.update(SD=Tw.T @ FD, eD=FD.T @ dw, QD=FD.T @ FD)
        return {a: torch.tensor(v) if isinstance(v, np.ndarray) else v for a, v in out.items()}

    def _spectra(self, th):
        """rho (C, ka), kappa (C, n, ka), kappa_dm (C, n, kd)."""
        case, C, n = self.case, th.shape[0], self.case["n_psr"]
        pc = math.log(YEAR ** 3 / (12.0 * math.pi ** 2) / self.d["tspan"])
        at, out = 0, []
        for K, m in ((case["nf_gw"], 1), (case["nf_rn"], n), (case["nf_dm"], n)):
            w = K if case["free"] else 2 if K else 0
            p = th[:, at:at + m * w].reshape(C, m, w)
            at += m * w
            if not K:
                v = th.new_zeros(C, m, 0)
            elif case["free"]:
                v = 10.0 ** p
            else:
                v = torch.exp(2.0 * LN10 * p[:, :, :1] - p[:, :, 1:] * self.lnfy[:K] + pc)
            out.append(v)
        wide = [torch.nn.functional.pad(v, (0, self.ka - v.shape[2])) for v in out[:2]]
        return wide[0][:, 0], wide[1], out[2]

    def logp(self, x, beta):
        th, u, z = _widths(self.case)
        spec = self._spectra(x[:, :th])
        cw = x[:, th:th + 8] if self.case["cw"] else None
        th += 8 * self.case["cw"]
        if self.case["form"] == "toa":
            return self._toa(spec, cw, x[:, th:th + u], x[:, th + u:]), None
        return self._std(spec, cw, x[:, th:], beta)

    def _toa(self, spec, cw, u, z):
        n, C, ka, kd = self.case["n_psr"], u.shape[0], self.ka, self.kd
        rho, kap, kdm = spec
        za, zd = z[:, :n * 2 * ka].reshape(C, n, ka, 2), z[:, n * 2 * ka:].reshape(C, n, kd, 2)
        phi = rho[:, :, None, None] * self.gamma + torch.diag_embed(kap.transpose(1, 2))
        a = torch.matmul(torch.linalg.cholesky(phi), za.transpose(1, 2).contiguous()).transpose(1, 2)
        ad = torch.sqrt(kdm)[..., None] * zd
        a = torch.cat([a.reshape(C, n, 2 * ka), ad.reshape(C, n, 2 * kd)], dim=2)
        b = self.d["sigma_b"] * u.reshape(C, n, 3)
        out = -0.5 * ((u * u).sum(1) + (z * z).sum(1) + (u.shape[1] + z.shape[1]) * LN2PI) - self.box
        for i, p in enumerate(self.psr):
            r = p["dt"] - a[:, i] @ p["T"].T - b[:, i] @ p["M"].T
            if cw is not None:
                r = r - _cw_delay(cw, p["t"], self.d["psr_pos"][i])
            out = out - 0.5 * ((r * r / p["N"]).sum(1) + torch.log(p["N"]).sum() + p["N"].numel() * LN2PI)
        return out

    def _data(self, cw, C):
        """d and dt^T N~^-1 dt per pulsar, of the data less the continuous wave."""
        if cw is None:
            return [(p["d"].expand(C, -1), p["c"]) for p in self.psr]
        K = self.case["cw_nf"]
        M = 2 * K + 1
        t = torch.arange(M, dtype=torch.float64) * (self.d["cw_tspan"] / M)
        arg = 2.0 * np.pi * np.outer(np.arange(1, K + 1), np.arange(M)) / M
        D = torch.tensor(np.stack([np.sin(arg), np.cos(arg)], axis=1).reshape(2 * K, M) * (2.0 / M))
        out = []
        for i, p in enumerate(self.psr):
            a = _cw_delay(cw, t, self.d["psr_pos"][i]) @ D.T
            out.append((p["d"] - a @ p["SD"].T, p["c"] - 2.0 * (a @ p["eD"]) + ((a @ p["QD"]) * a).sum(1)))
        return out

    @staticmethod
    def _factor(S0, v, beta):
        """Lower Cholesky factor of the precision in reversed order: L = flip(its inverse transposed)."""
        A = beta[:, None, None] * S0 + torch.diag_embed(1.0 / v)
        return torch.linalg.cholesky(torch.flip(A, (1, 2)))

    @staticmethod
    def _solve(L, y, upper):
        m = L.transpose(1, 2) if upper else L
        return torch.linalg.solve_triangular(m, y[..., None], upper=upper)[..., 0]

    def _std(self, spec, cw, z, beta):
        case, n, C, ka, kd, kg, kr = (self.case, self.case["n_psr"], z.shape[0], self.ka, self.kd,
                                      self.case["nf_gw"], self.case["nf_rn"])
        rho, kap, kdm = spec
        z = z.reshape(C, n, -1)
        data = self._data(cw, C)
        two = lambda v: v.repeat_interleave(2, dim=-1)  # noqa: E731
        out, coef, parts = z.new_zeros(C) - self.box, [], []
        for i, p in enumerate(self.psr):
            dv, cv = data[i]
            D = torch.cat([two(rho + kap[:, i]), two(kdm[:, i])], dim=1)
            L = self._factor(p["S0"], D, beta)
            t = self._solve(L, torch.flip(beta[:, None] * dv, (1,)), False)
            if not case["split"]:
                a = torch.flip(self._solve(L, t + torch.flip(z[:, i], (1,)), True), (1,))
                out = out - torch.log(torch.diagonal(L, dim1=1, dim2=2)).sum(1)
                coef.append(a)
            else:
                ah = torch.flip(self._solve(L, t, True), (1,))
                g, r = list(range(2 * kg)), list(range(2 * kr)) + list(range(2 * ka, 2 * ka + 2 * kd))
                a, pair = torch.zeros_like(ah), []
                for rows, v, zz in ((g, two(rho[:, :kg]), z[:, i, :2 * kg]),
                                    (r, torch.cat([two(kap[:, i, :kr]), two(kdm[:, i])], dim=1), z[:, i, 2 * kg:])):
                    Lb = self._factor(p["S0"][rows][:, rows], v, beta)
                    ab = v / D[:, rows] * ah[:, rows] + torch.flip(self._solve(Lb, torch.flip(zz, (1,)), True), (1,))
                    out = out - torch.log(torch.diagonal(Lb, dim1=1, dim2=2)).sum(1)
                    a = a.index_add(1, torch.tensor(rows), ab)
                    pair.append(ab)
                out = out - 0.5 * (pair[1] ** 2 / v + torch.log(2.0 * math.pi * v)).sum(1)
                parts.append(pair[0])
                coef.append(torch.cat(pair, dim=1))
            out = out + beta * (p["k"] - 0.5 * cv + (a * dv).sum(1) - 0.5 * ((a @ p["S0"]) * a).sum(1))
        a = torch.stack(coef, dim=1)
        # prior of the common rows: dense over the pulsars, sin and cos alike
        if case["split"]:
            L, y = torch.linalg.cholesky(self.gamma), torch.stack(parts, dim=1)
            y = torch.linalg.solve_triangular(L, y.contiguous(), upper=False)
            out = out - 0.5 * (y * y / two(rho[:, None, :kg])).sum((1, 2)) - kg * n * LN2PI
            out = out - n * torch.log(rho[:, :kg]).sum(1) - 2 * kg * torch.log(torch.diagonal(L)).sum()
        else:
            phi = rho[:, :kg, None, None] * self.gamma + torch.diag_embed(kap[:, :, :kg].transpose(1, 2))
            L = torch.linalg.cholesky(phi)
            y = a[:, :, :2 * kg].reshape(C, n, kg, 2).transpose(1, 2).contiguous()
            y = torch.linalg.solve_triangular(L, y, upper=False)
            out = out - 0.5 * (y * y).sum((1, 2, 3)) - kg * n * LN2PI
            out = out - 2.0 * torch.log(torch.diagonal(L, dim1=2, dim2=3)).sum((1, 2))
            for v, w in ((two(kap[:, :, kg:]), a[:, :, 2 * kg:2 * ka]), (two(kdm), a[:, :, 2 * ka:])):
                out = out - 0.5 * (w * w / v + torch.log(2.0 * math.pi * v)).sum((1, 2))
        return out, a

    def __call__(self, x, beta):
        """(logp, grad, coefficients) of points x (C, d) as tensors, a few chains at a time."""
        got = []
        for c in range(0, x.shape[0], 8):
            xs = torch.tensor(x[c:c + 8], requires_grad=True)
            bs = torch.ones(xs.shape[0], dtype=torch.float64) if beta is None else torch.tensor(beta[c:c + 8])
            lp, a = self.logp(xs, bs)
            (gr,) = torch.autograd.grad(lp.sum(), xs)
            got.append((lp.detach(), gr, torch.zeros(0) if a is None else a.detach()))
        return [torch.cat(v) for v in zip(*got)]


def _philox(index, chain, traj, purpose):
    """Philox4x32-10 (Salmon et al., SC'11) of the counter (index, chain, traj, purpose) with the key SEED."""
    c = [np.asarray(v, np.uint64) for v in np.broadcast_arrays(index, chain, traj, purpose)]
    k, low = [SEED & 0xFFFFFFFF, SEED >> 32], np.uint64(0xFFFFFFFF)
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k[0]), p1 & low, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k[1]),
             p0 & low]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    u = [((a << np.uint64(21)) | (b >> np.uint64(11))).astype(np.float64) for a, b in ((c[0], c[1]), (c[2], c[3]))]
    return (u[0] + 1.0) * 2.0 ** -53, u[1] * 2.0 ** -53


def _trajectory(case, ref, x, beta):
    """The first trajectory from x: momenta, leapfrog and the accept test."""
    C, d = x.shape
    im, eps = _inv_mass(case, d), _eps(case)
    u1, u2 = _philox(np.arange((d + 1) // 2)[None, :], np.arange(C)[:, None], 0, 0)
    r = np.sqrt(-2.0 * np.log(u1))
    p = np.stack([r * np.cos(2.0 * np.pi * u2), r * np.sin(2.0 * np.pi * u2)], axis=2).reshape(C, -1)[:, :d]
    p = p / np.sqrt(im)
    lp0, g0 = (v.numpy() for v in ref(x, beta)[:2])
    h0 = -lp0 + 0.5 * np.sum(im * p * p, axis=1)
    xn, p = x.copy(), p + 0.5 * eps * g0
    for step in range(case["leapfrog"]):
        xn = xn + eps * im * p
        lp, g = (v.numpy() for v in ref(xn, beta)[:2])
        p = p + (eps if step + 1 < case["leapfrog"] else 0.5 * eps) * g
    h1 = -lp + 0.5 * np.sum(im * p * p, axis=1)
    ok = np.log(_philox(0, np.arange(C), 0, 1)[0]) < h0 - h1
    return dict(x=np.where(ok[:, None], xn, x), logp=np.where(ok, lp, lp0), grad=np.where(ok[:, None], g, g0),
                accept=None)


def exact(case, seed):
    w = work(case)["flops"]
    if w > (2e10 if case["call"] == "hmc" else 4e10):      # many seconds on the CPU
        return None
    d = _array(case, seed)
    x, beta = _points(case, seed)
    ref = _Reference(case, d)
    if case["call"] == "hmc":
        return _trajectory(case, ref, x, beta)
    logp, grad, coef = ref(x, beta)
    out = dict(logp=logp, grad=grad, status=None)
    if case["call"] == "coef":
        out["coef"] = coef
    return out
