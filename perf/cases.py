"""The workloads the library is timed on: what a reacting-flow program calls,
through the Python binding, at the sizes it calls it with.

A case is a dict of plain values:

  op         rates      net production rates
             step       rates, then transport: what an explicit step asks for
             transport  mixture-averaged mu, lambda, D_km
             thermo     cp_k, h_k, cp
             jacobian   d wdot / d C, one matrix per point
             qss        rates of a mechanism with quasi-steady-state species
             batch      rates and transport of several point sets in one call
  ns, nr     species and reactions (the seeded synthetic mechanisms of
             paper_2411_02640_amd.inputs; 9/21, 53/325 and 200/1500 are the
             named ones)
  n          grid points (of all point sets together, for a batch)
  precision  fp64 or mixed (rates, step, transport, batch)
  dkj        the diffusion tables hold fits of D_kj instead of 1/D_kj
  forms      part of the reactions are SRI, chemically activated or PLOG
  items      point sets of a batch

prepare() makes the device mechanism and the states: T ~ U[300, 2800] K,
p ~ U[1, 40] atm, Y ~ Dirichlet(0.3).  exact() evaluates the same formulas
(arXiv 2411.02640, App. A) reaction by reaction in plain torch float64.
"""
import functools
import math

import numpy as np
import torch

from paper_2411_02640_amd import inputs, kx, opcount

DEVICE = "cuda:0"
R_GAS = 8.31446261815324e7      # erg / (mol K)
R_CAL = 8.31446261815324 / 4.184
P_ATM = 1013250.0


def listed():
    return [
        # the small mechanism on the block of points one rank of a small domain
        # holds: a call of a few microseconds of work, so latency counts
        dict(name="step_9sp_4k", op="step", ns=9, nr=21, n=4096, precision="fp64"),
        # a 53-species solver block (one element patch) with the reaction forms
        # of imported mechanisms; far from filling the GPU
        dict(name="step_53sp_forms_2k", op="step", ns=53, nr=325, n=2011, precision="fp64",
             forms=True),
        # the benchmark's workload, its two kernels by themselves
        dict(name="rates_53sp_1m", op="rates", ns=53, nr=325, n=1 << 20, precision="fp64"),
        dict(name="transport_53sp_1m", op="transport", ns=53, nr=325, n=1 << 20,
             precision="fp64"),
        # the mixed-precision path on a domain of a quarter million points (odd)
        dict(name="step_53sp_mixed_250k", op="step", ns=53, nr=325, n=250001,
             precision="mixed"),
        # a large mechanism on an ordinary domain (ragged)
        dict(name="rates_200sp_100k", op="rates", ns=200, nr=1500, n=100003, precision="fp64"),
        dict(name="transport_200sp_100k", op="transport", ns=200, nr=1500, n=100003,
             precision="fp64"),
        # tables that hold D_kj itself, the form of the paper's equation
        dict(name="transport_53sp_dkj_300k", op="transport", ns=53, nr=325, n=300007,
             precision="fp64", dkj=True),
        # mixture thermodynamics beside every step
        dict(name="thermo_53sp_1m", op="thermo", ns=53, nr=325, n=1 << 20),
        # Jacobians for an implicit integrator's Newton steps
        dict(name="jacobian_53sp_32k", op="jacobian", ns=53, nr=325, n=1 << 15),
        # a reduced mechanism: 6 of 53 species quasi-steady
        dict(name="qss_53sp_256k", op="qss", ns=53, nr=325, n=1 << 18),
        # a solver's blocks of different sizes in one call
        dict(name="batch_53sp_8x", op="batch", ns=53, nr=325, n=60013, items=8,
             precision="fp64"),
    ]


def draw(rng):
    op = rng.choice(["rates", "step", "transport", "thermo", "jacobian", "qss", "batch"])

    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    if op == "qss":
        return dict(op=op, ns=53, nr=325, n=log_int(1000, 1 << 18),
                    **({"forms": True} if rng.random() < 0.3 else {}))
    ns = rng.choice([9, 53, log_int(17, 100), log_int(17, 200), 200])
    if op == "jacobian":
        ns = min(ns, 100)
    nr = {9: 21, 53: 325, 200: 1500}.get(ns, 7 * ns)
    # no case costs more than the largest listed one of its kind
    cap = {"rates": (325 << 20) // nr, "step": (325 << 18) // nr, "batch": 325 * 60013 // nr,
           "transport": 53 * (53 << 20) // ns ** 2, "thermo": (53 << 20) // ns,
           "jacobian": 53 * (53 << 15) // ns ** 2}[op]
    if op in ("step", "batch"):
        cap = min(cap, 53 * (53 << 18) // ns ** 2)
    case = dict(op=op, ns=ns, nr=nr)
    if op == "transport" and rng.random() < 0.3:
        case["dkj"] = True
        cap //= 4
    case["n"] = log_int(256, min(1 << 20, cap))
    if op in ("rates", "step", "transport", "batch"):
        case["precision"] = rng.choice(["fp64", "fp64", "mixed"])
    if op == "batch":
        case["items"] = rng.randint(2, 32)
    if ns == 53 and op in ("rates", "step", "jacobian") and rng.random() < 0.3:
        case["forms"] = True
    return case


@functools.lru_cache(maxsize=None)
def _mechanism(ns, nr, qss, dkj, forms):
    """The mechanism's tables as a program reads them from its files, once."""
    named = {(9, 21): inputs.MECH_9, (53, 325): inputs.MECH_53, (200, 1500): inputs.MECH_200}
    spec = named.get((ns, nr))
    kw = {}
    if spec is None:
        falloff, three, lind = max(1, nr * 6 // 100), max(1, nr // 10), nr // 50
        kw.update(n_species=ns, n_elementary=nr - falloff - three - lind, n_threebody=three,
                  n_lindemann=lind, n_troe=falloff, seed=9000 + ns)
    else:
        kw.update(n_species=ns, n_elementary=spec.n_elementary, n_threebody=spec.n_threebody,
                  n_lindemann=spec.n_lindemann, n_troe=spec.n_troe, seed=spec.seed)
    if forms:
        kw.update(n_sri=10, n_chemact=8, n_plog=20)
    if qss:
        kw.update(n_qss=6)
    if dkj:
        kw.update(diff_fit_kind=0)
    return inputs.make_mechanism(inputs.MechSpec(**kw))


def _mech(case):
    return _mechanism(case["ns"], case["nr"], case["op"] == "qss", bool(case.get("dkj")),
                      bool(case.get("forms")))


def _sizes(case):
    """Points of each set: one, or a batch's sets of uneven sizes."""
    n, items = case["n"], case.get("items", 1)
    w = [1.0 + (i * i) % 7 for i in range(items)]
    sizes = [max(1, int(n * x / sum(w))) for x in w]
    sizes[-1] += n - sum(sizes)
    return sizes


def _states(case, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    kw = dict(dtype=torch.float64, device=DEVICE)
    out = []
    for n in _sizes(case):
        T = 300.0 + 2500.0 * torch.rand(n, generator=g, **kw)
        p = P_ATM * (1.0 + 39.0 * torch.rand(n, generator=g, **kw))
        gam = torch._standard_gamma(torch.full((case["ns"], n), 0.3, **kw), generator=g)
        out.append((T, p, (gam / gam.sum(0, keepdim=True)).contiguous()))
    return out


def prepare(case, seed):
    return {"op": case["op"], "precision": case.get("precision", "fp64"),
            "mech": kx.Mechanism(_mech(case), 0), "sets": _states(case, seed)}


def run(state):
    op, dm, prec = state["op"], state["mech"], state["precision"]
    if op == "batch":
        return kx.batch_noalloc(dm, state["sets"], transport=True, precision=prec)
    (T, p, Y), = state["sets"]
    if op == "rates" or op == "qss":
        return kx.production_rates(dm, T, p, Y, precision=prec)
    if op == "transport":
        return kx.transport(dm, T, p, Y, precision=prec)
    if op == "step":
        return (kx.production_rates(dm, T, p, Y, precision=prec),
                *kx.transport(dm, T, p, Y, precision=prec))
    if op == "thermo":
        return kx.thermo(dm, T, Y)
    return kx.jacobian(dm, T, p, Y)


def work(case):
    m, n, ns, op = _mech(case), case["n"], case["ns"], case["op"]
    per, io = opcount.per_point(m), opcount.io_bytes(m)
    rates, trans = float(per["rates_flops"]), float(per["transport_flops"])
    flops, nbytes = {
        "rates": (rates, io["rates"]),
        "qss": (rates, io["rates"]),
        "transport": (trans, io["transport"]),
        "step": (rates + trans, io["fused"]),
        "batch": (rates + trans, io["fused"]),
        "thermo": (20 * ns, 8 * (3 * ns + 2)),
        # every reaction's slot derivatives into the rows of its species
        "jacobian": (rates + 40 * case["nr"], 8 * (ns * ns + ns + 2)),
    }[op]
    return {"bytes": nbytes * n, "flops": flops * n}


# --------------------------------------------------------------------------
# the same quantities in plain torch float64
# --------------------------------------------------------------------------
def _gibbs(m, T):
    """G_k / RT = H/RT - S/R from the NASA-7 polynomials, [ns][n]."""
    out = []
    lnT = torch.log(T)
    for k in range(m["n_species"]):
        g = []
        for a in (m["nasa_lo"][k], m["nasa_hi"][k]):
            h = (a[0] + a[1] * T / 2 + a[2] * T**2 / 3 + a[3] * T**3 / 4 + a[4] * T**4 / 5
                 + a[5] / T)
            s = a[0] * lnT + a[1] * T + a[2] * T**2 / 2 + a[3] * T**3 / 3 + a[4] * T**4 / 4 + a[6]
            g.append(h - s)
        out.append(torch.where(T < m["t_mid"][k], g[0], g[1]))
    return out


def _arrhenius(A, beta, Ea, T):
    return A * torch.exp(beta * torch.log(T) - (Ea / R_CAL) / T)


def _log10(x):
    return torch.log10(torch.clamp(x, min=np.finfo(float).tiny))


def _side(m, which, i):
    ptr, sp, nu = m[which + "_ptr"], m[which + "_sp"], m[which + "_nu"]
    return [(int(sp[e]), int(nu[e])) for e in range(ptr[i], ptr[i + 1])]


def _net(m, i):
    net = {}
    for k, v in _side(m, "reac", i):
        net[k] = net.get(k, 0) - v
    for k, v in _side(m, "prod", i):
        net[k] = net.get(k, 0) + v
    return {k: v for k, v in net.items() if v}


class _Point:
    """Concentrations and per-reaction factors at a set of points."""

    def __init__(self, m, T, p, Y):
        ns = m["n_species"]
        W = np.asarray(m["composition"], dtype=np.float64) @ m["elem_mass"]
        qss = m["qss"] if m.get("qss") is not None else np.zeros(ns, np.int32)
        self.m, self.T, self.p, self.qss = m, T, p, qss
        self.M = p / (R_GAS * T)
        wsum = sum(Y[k] / W[k] for k in range(ns) if not qss[k])
        self.C = [self.M * (Y[k] / W[k]) / wsum if not qss[k] else None for k in range(ns)]
        self.g = _gibbs(m, T)

    def third_body(self, i):
        m = self.m
        X = m["eff_default"][i] * self.M
        for e in range(m["eff_ptr"][i], m["eff_ptr"][i + 1]):
            X = X + (m["eff_val"][e] - m["eff_default"][i]) * self.C[int(m["eff_sp"][e])]
        return X

    def plog(self, i):
        m = self.m
        j0, j1 = int(m["plog_ptr"][i]), int(m["plog_ptr"][i + 1])
        ln = [torch.log(_arrhenius(m["plog_A"][j], m["plog_beta"][j], m["plog_Ea"][j], self.T))
              for j in range(j0, j1)]
        lp = [math.log(m["plog_p"][j]) for j in range(j0, j1)]
        lnp = torch.log(self.p)
        val, slope = ln[0], torch.zeros_like(lnp)
        for j in range(len(ln) - 1):
            s = (ln[j + 1] - ln[j]) / (lp[j + 1] - lp[j])
            inside = lnp > lp[j]
            val = torch.where(inside, ln[j] + s * (lnp - lp[j]), val)
            slope = torch.where(inside, s, slope)
        above = lnp >= lp[-1]
        return (torch.exp(torch.where(above, ln[-1], val)),
                torch.where(above, torch.zeros_like(slope), slope))

    def blend(self, i, Pr):
        """F of eq:blend and d ln F / d ln P_r."""
        m, T = self.m, self.T
        lp = _log10(Pr)
        if m["rxn_type"][i] == 3:
            al, T3, T1, T2 = m["troe"][i]
            Fc = (1 - al) * torch.exp(-T / T3) + al * torch.exp(-T / T1)
            if not np.isnan(T2):
                Fc = Fc + torch.exp(-T2 / T)
            lF = _log10(Fc)
            x, nn = lp - 0.4 - 0.67 * lF, 0.75 - 1.27 * lF
            f1 = x / (nn - 0.14 * x)
            F = 10.0 ** (lF / (1 + f1 * f1))
            return F, -2.0 * lF * f1 / (1 + f1 * f1) ** 2 * nn / (nn - 0.14 * x) ** 2
        if m["rxn_type"][i] == 4:
            a, b, c, d, e = m["sri"][i]
            X = 1.0 / (1.0 + lp * lp)
            B = a * torch.exp(-b / T) + torch.exp(-T / c)
            return (d * B ** X * T ** e,
                    -2.0 * torch.log(B) * lp * X * X / math.log(10.0))
        return torch.ones_like(T), torch.zeros_like(T)

    def reaction(self, i, slopes=False):
        """k_f, k_r, c_i (and dc/d[X], d ln k_f / d ln p) of reaction i."""
        m, T = self.m, self.T
        t = int(m["rxn_type"][i])
        slope = dc = None
        if t == 5:
            kf, slope = self.plog(i)
        else:
            kf = _arrhenius(m["A"][i], m["beta"][i], m["Ea"][i], T)
        c = torch.ones_like(T)
        if t == 1:
            c = self.third_body(i)
            dc = torch.ones_like(T)
        elif t in (2, 3, 4):
            X = self.third_body(i)
            k0 = _arrhenius(m["A0"][i], m["beta0"][i], m["Ea0"][i], T)
            e0 = k0 / kf
            Pr = e0 * X
            F, g = self.blend(i, Pr)
            if m.get("chem_act") is not None and m["chem_act"][i]:
                c, kf = F / (1 + Pr), k0
                if slopes:
                    dc = F * (g / (X * (1 + Pr)) - e0 / (1 + Pr) ** 2)
            else:
                c = Pr / (1 + Pr) * F
                if slopes:
                    dc = e0 * F * (1 / (1 + Pr) ** 2 + g / (1 + Pr))
        kr = None
        if m["reversible"][i]:
            net = _net(m, i)
            dG = sum(v * self.g[k] for k, v in net.items()) if net else torch.zeros_like(T)
            kr = kf * torch.exp(dG) * (P_ATM / (R_GAS * T)) ** (-sum(net.values()))
        return kf, kr, c, dc, slope


def _product(C, side):
    out = 1.0
    for k, v in side:
        for _ in range(v):
            out = out * C[k]
    return out


def _exact_rates(m, T, p, Y):
    P = _Point(m, T, p, Y)
    ns, nr = m["n_species"], m["n_reactions"]
    C = list(P.C)
    if P.qss.any():
        # the balances of the quasi-steady species are linear in their
        # concentrations: at most one such molecule on a side
        q = [k for k in range(ns) if P.qss[k]]
        at = {k: j for j, k in enumerate(q)}
        A = torch.zeros((T.numel(), len(q), len(q)), dtype=T.dtype, device=T.device)
        b = torch.zeros((T.numel(), len(q)), dtype=T.dtype, device=T.device)
        for i in range(nr):
            net = {k: v for k, v in _net(m, i).items() if k in at}
            if not net:
                continue
            kf, kr, c, _, _ = P.reaction(i)
            for k_side, sign, which in ((kf, 1.0, "reac"), (kr, -1.0, "prod")):
                if k_side is None:
                    continue
                side = _side(m, which, i)
                term = sign * c * k_side * _product(C, [s for s in side if s[0] not in at])
                col = [at[k] for k, _ in side if k in at]
                for k, v in net.items():
                    if col:
                        A[:, at[k], col[0]] += v * term
                    else:
                        b[:, at[k]] += v * term
        x = torch.linalg.solve(A, -b.unsqueeze(-1)).squeeze(-1)
        for j, k in enumerate(q):
            C[k] = x[:, j]
    wdot = torch.zeros_like(Y)
    for i in range(nr):
        kf, kr, c, _, _ = P.reaction(i)
        R = kf * _product(C, _side(m, "reac", i))
        if kr is not None:
            R = R - kr * _product(C, _side(m, "prod", i))
        R = R * c
        for k, v in _net(m, i).items():
            if not P.qss[k]:
                wdot[k] += v * R
    return wdot


def _exact_jacobian(m, T, p, Y):
    P = _Point(m, T, p, Y)
    ns = m["n_species"]
    J = torch.zeros((ns, ns, T.numel()), dtype=T.dtype, device=T.device)
    for i in range(m["n_reactions"]):
        kf, kr, c, dc, slope = P.reaction(i, slopes=True)
        sides = [(kf, 1.0, _side(m, "reac", i))]
        if kr is not None:
            sides.append((kr, -1.0, _side(m, "prod", i)))
        net = _net(m, i)
        grad, q = {}, 0.0
        for kk, sign, side in sides:
            q = q + sign * kk * _product(P.C, side)
            for j, v in side:
                rest = [(k, u - (k == j)) for k, u in side]
                d = sign * v * c * kk * _product(P.C, rest)
                grad[j] = grad[j] + d if j in grad else d
        dense = None
        if dc is not None:
            D = dc * q
            dense = m["eff_default"][i] * D
            for e in range(m["eff_ptr"][i], m["eff_ptr"][i + 1]):
                j = int(m["eff_sp"][e])
                d = D * (m["eff_val"][e] - m["eff_default"][i])
                grad[j] = grad[j] + d if j in grad else d
        if slope is not None:
            d = c * q * slope / P.M
            dense = d if dense is None else dense + d
        for k, v in net.items():
            if dense is not None:
                J[k] += v * dense
            for j, d in grad.items():
                J[k, j] += v * d
    return J.permute(2, 0, 1).contiguous()


def _poly(c, u):
    return sum(c[..., o] * u ** o for o in range(c.shape[-1]))


def _exact_transport(m, T, p, Y):
    kw = dict(dtype=T.dtype, device=T.device)
    W = torch.as_tensor(np.asarray(m["composition"], dtype=np.float64) @ m["elem_mass"], **kw)
    ns = m["n_species"]
    u = (torch.log(T) - m["fit_L0"]) / m["fit_h"]
    fits = [torch.as_tensor(m[f], **kw) for f in ("visc_fit", "cond_fit", "diff_fit")]
    X = Y / W[:, None]
    X = X / X.sum(0)
    wbar = (X * W[:, None]).sum(0)
    eta = _poly(fits[0][:, None, :], u)
    cond = _poly(fits[1][:, None, :], u)
    lam = 0.5 * ((X * cond).sum(0) + 1.0 / (X / cond).sum(0))
    mu = torch.zeros_like(T)
    D = torch.empty_like(Y)
    for k in range(ns):
        t = 1.0 + torch.sqrt(eta[k] / eta) * (W / W[k])[:, None] ** 0.25
        phi = t * t / torch.sqrt(8.0 * (1.0 + W[k] / W))[:, None]
        mu += X[k] * eta[k] / (X * phi).sum(0)
        f = _poly(fits[2][k][:, None, :], u)
        g = X * f if m["diff_fit_kind"] == 1 else X / f
        S = torch.cat([g[:k], g[k + 1:]]).sum(0)
        D[k] = (wbar - X[k] * W[k]) / wbar / S * (P_ATM / p)
    return mu, lam, D


def _exact_thermo(m, T, Y):
    W = np.asarray(m["composition"], dtype=np.float64) @ m["elem_mass"]
    cps, hs, cp = [], [], 0.0
    for k in range(m["n_species"]):
        lo = T < m["t_mid"][k]
        c, h = [], []
        for a in (m["nasa_lo"][k], m["nasa_hi"][k]):
            c.append(a[0] + a[1] * T + a[2] * T**2 + a[3] * T**3 + a[4] * T**4)
            h.append(a[0] * T + a[1] * T**2 / 2 + a[2] * T**3 / 3 + a[3] * T**4 / 4
                     + a[4] * T**5 / 5 + a[5])
        cps.append(torch.where(lo, c[0], c[1]) * (R_GAS / W[k]))
        hs.append(torch.where(lo, h[0], h[1]) * (R_GAS / W[k]))
        cp = cp + Y[k] * cps[-1]
    return torch.stack(cps), torch.stack(hs), cp


def _in_chunks(f, arrays, size, dim=-1):
    """f over the points in pieces, joined again along the points."""
    n = arrays[0].shape[-1]
    parts = [f(*[a[..., i:i + size].contiguous() for a in arrays]) for i in range(0, n, size)]
    if isinstance(parts[0], torch.Tensor):
        return torch.cat(parts, dim=dim)
    return tuple(torch.cat([q[j] for q in parts], dim=dim) for j in range(len(parts[0])))


def exact(case, seed):
    m, op = _mech(case), case["op"]
    # the points of a piece: as many as keep the temporaries within a few GB
    size = max(1024, (1 << 26) // (case["ns"] * (case["ns"] if op == "jacobian" else 4)))
    rates = functools.partial(_exact_rates, m)
    trans = functools.partial(_exact_transport, m)
    out = []
    for T, p, Y in _states(case, seed):
        if op in ("rates", "qss"):
            return _in_chunks(rates, (T, p, Y), size)
        if op == "transport":
            return _in_chunks(trans, (T, p, Y), size)
        if op == "thermo":
            return _in_chunks(functools.partial(_exact_thermo, m), (T, Y), size)
        if op == "jacobian":
            return _in_chunks(functools.partial(_exact_jacobian, m), (T, p, Y), size, dim=0)
        out.append((_in_chunks(rates, (T, p, Y), size), *_in_chunks(trans, (T, p, Y), size)))
    return out[0] if op == "step" else out
