"""The work a user has this library do, as cases that can be timed and compared.

Each case is one call (or one whole batch, or a few PIC steps) through the
package's public entry points at a size that the repository's own workloads,
tests and benchmark use, or an odd size between them: the CV scan over a list
of concentrations, its first-order (triangle) form, the refined minimiser,
the deposit and the gather with one or per-particle concentrations, the two
adaptive width rules, a batch of whole solves, and resident PIC sessions, in
double and in float. ``exact`` evaluates the definitions directly in 64 bits
with torch.
"""
import math

import numpy as np
import torch

import paper_1804_11174_amd as kde

DEV = "cuda"
F64, F32 = torch.float64, torch.float32


# ----------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest scan that users run: 4096 particles, 8 concentrations; launches and latency
        {"name": "scan_small_f64", "kind": "scan", "dtype": "f64", "n": 4096, "B": 8, "k_lo": 1.0, "k_hi": 1e3,
         "amp": 0.1, "mode": 1},
        # paper scale: the 65,536-particle subsample over 32 concentrations
        {"name": "scan_paper_f64", "kind": "scan", "dtype": "f64", "n": 65536, "B": 32, "k_lo": 1.0, "k_hi": 1e4,
         "amp": 0.5, "mode": 1},
        # a served request's scan in float, an odd count, 16 concentrations
        {"name": "scan_request_f32", "kind": "scan", "dtype": "f32", "n": 20011, "B": 16, "k_lo": 1.0, "k_hi": 1e4,
         "amp": 0.2, "mode": 1},
        # the first-order shape's scan over half-widths from a quarter cell to half the period
        {"name": "tri_scan_f64", "kind": "tri_scan", "dtype": "f64", "n": 30001, "B": 32, "M": 256, "amp": 0.5,
         "mode": 1},
        # the refined concentration of the paper-scale set (moments, series, Newton)
        {"name": "refine_f64", "kind": "refine", "dtype": "f64", "n": 65536, "B": 32, "k_lo": 1.0, "k_hi": 1e4,
         "amp": 0.5, "mode": 1},
        # the pilot density of a paper-scale set: one concentration, 1,048,576 particles on 256 nodes
        {"name": "pilot_deposit_f64", "kind": "deposit", "dtype": "f64", "shape": "vm", "n": 1048576, "M": 256,
         "kappa": 26.263635276533325, "per": False, "amp": 0.5, "mode": 1},
        # a PIC step's deposit with per-particle concentrations in float, odd count
        {"name": "adaptive_deposit_f32", "kind": "deposit", "dtype": "f32", "shape": "vm", "n": 262147, "M": 128,
         "kappa": 10.0, "per": True, "amp": 0.3, "mode": 1},
        # the field gathered back to a paper-scale set with per-particle concentrations
        {"name": "adaptive_gather_f64", "kind": "gather", "dtype": "f64", "shape": "vm", "n": 1048576, "M": 256,
         "kappa": 26.263635276533325, "per": True, "amp": 0.5, "mode": 1},
        # Silverman's widths from the pilot grid: memory traffic
        {"name": "widths_f64", "kind": "widths", "dtype": "f64", "n": 1048576, "M": 256, "kappa": 26.263635276533325,
         "amp": 0.5, "mode": 1},
        # the widths from the pilot evaluated exactly at each particle, float positions, odd count
        {"name": "widths_exact_f32", "kind": "widths_exact", "dtype": "f32", "n": 1000003, "kappa": 24.65,
         "amp": 0.5, "mode": 1},
        # many small and middling solves at once (scan, pilot, widths, adaptive density), float
        {"name": "batch_f32", "kind": "batch", "dtype": "f32", "sets": 24, "n_lo": 1000, "n_hi": 30000, "B": 16},
        # a resident PIC session of the serving workload, a few steps between diagnostics
        {"name": "session_f32", "kind": "session", "dtype": "f32", "n": 262144, "M": 128, "steps": 4, "B": 16,
         "n_cv": 65536, "L": 4.0 * math.pi, "dt": 0.1, "amp": 0.01, "v_th": 1.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scan", "scan", "tri_scan", "refine", "deposit", "deposit", "gather", "gather", "widths",
                       "widths_exact", "batch", "session"])
    c = {"kind": kind, "dtype": rng.choice(["f64", "f32"])}
    if kind in ("batch", "session"):
        if kind == "batch":
            c.update(sets=_log_int(rng, 4, 32), n_lo=1000, n_hi=_log_int(rng, 3000, 30000), B=16)
        elif rng.random() < 0.5:
            c.update(n=_log_int(rng, 20000, 262144), M=rng.choice([64, 128, 256]), steps=rng.randint(1, 6), B=16,
                     n_cv=16384, L=4.0 * math.pi, dt=0.1, amp=0.01, v_th=1.0)
        else:  # the Landau ensembles' shape
            c.update(n=32768, M=256, steps=rng.randint(4, 12), B=16, n_cv=32768, L=2.0 * math.pi, dt=0.01, amp=0.02,
                     v_th=round(rng.uniform(0.2, 0.45), 3))
        return c
    c["amp"] = round(rng.uniform(0.01, 0.5), 4)
    c["mode"] = rng.choice([1, 1, 2, 4])
    if kind == "scan":
        c.update(n=_log_int(rng, 1000, 60000), B=rng.choice([8, 16, 24, 32]), k_lo=1.0,
                 k_hi=round(10.0 ** rng.uniform(2.5, 4.0), 3))
    elif kind == "tri_scan":
        c.update(n=_log_int(rng, 1000, 50000), B=rng.choice([8, 16, 32]), M=rng.choice([64, 128, 256]))
    elif kind == "refine":
        c.update(n=_log_int(rng, 1000, 200000), B=rng.choice([8, 16, 32]), k_lo=1.0,
                 k_hi=round(10.0 ** rng.uniform(2.5, 4.0), 3))
    elif kind in ("deposit", "gather"):
        shape = rng.choice(["vm", "vm", "tri"])
        c.update(shape=shape, n=_log_int(rng, 2000, 1048576), M=rng.choice([64, 100, 128, 256, 300, 512]),
                 per=rng.random() < 0.6, kappa=round(10.0 ** rng.uniform(0.3, 3.0), 4))
    elif kind == "widths":
        c.update(n=_log_int(rng, 2000, 1048576), M=rng.choice([64, 128, 256, 300]),
                 kappa=round(10.0 ** rng.uniform(0.3, 2.5), 4))
    else:
        c.update(n=_log_int(rng, 2000, 1048576), kappa=round(10.0 ** rng.uniform(0.3, 2.5), 4))
    return c


# ------------------------------------------------------------------ inputs

def _dtype(c):
    return F64 if c["dtype"] == "f64" else F32


def _period(c):
    return 4.0 * math.pi


def _rng(seed, part=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + 17 + part)
    return g


def _positions(seed, n, L, amp, mode, dtype, part=0):
    """n draws on [0, L) of (1 + amp cos(k x)) / L, k = 2 pi mode / L: the distribution function solved for x."""
    u = torch.rand(n, dtype=F64, device=DEV, generator=_rng(seed, part)) * L
    k = 2.0 * math.pi * mode / L
    x = u.clone()
    for _ in range(60):
        x = u - (amp / k) * torch.sin(k * x)
    x = torch.remainder(x, L).to(dtype)
    return torch.where(x >= L, torch.zeros_like(x), x).contiguous()


def _log_list(lo, hi, count):
    return np.geomspace(lo, hi, count)


def _density(x, L, amp, mode):
    return (1.0 + amp * torch.cos((2.0 * math.pi * mode / L) * x.to(F64))) / L


def _half_width(c, L):
    """The triangle's half-width of a case: as wide as the von Mises kernel of its concentration, within [L/M, L/4]."""
    return min(max(L / (2.0 * math.pi * math.sqrt(c["kappa"])), L / c["M"]), 0.25 * L)


def _per_particle(c, x, L):
    """Silverman's concentrations (half-widths for the triangle) for positions drawn from the case's density."""
    f = _density(x, L, c["amp"], c["mode"])
    ratio = f / torch.exp(torch.log(f).mean())
    if c["shape"] == "tri":
        return (_half_width(c, L) / torch.sqrt(ratio)).clamp(max=0.45 * L).to(x.dtype).contiguous()
    return (c["kappa"] * ratio).to(x.dtype).contiguous()


def _field(seed, M, L):
    """A grid field as a PIC step has it: a few modes and noise."""
    x = torch.arange(M, dtype=F64, device=DEV) * (2.0 * math.pi / M)
    a = torch.randn(4, 2, dtype=F64, device=DEV, generator=_rng(seed, 5))
    e = sum((a[m, 0] * torch.cos((m + 1) * x) + a[m, 1] * torch.sin((m + 1) * x)) / (m + 1) for m in range(4))
    return (e + 0.05 * torch.randn(M, dtype=F64, device=DEV, generator=_rng(seed, 6))).contiguous()


def _batch_sets(c, seed):
    r = np.random.default_rng([c["sets"], c["n_lo"], c["n_hi"]])  # the sets' sizes are the case's, the positions the seed's
    out = []
    for s in range(c["sets"]):
        n = int(round(math.exp(r.uniform(math.log(c["n_lo"]), math.log(c["n_hi"])))))
        amp, k, M = float(r.uniform(0.01, 0.5)), float(r.choice([0.5, 1.0, 2.0])), int(r.choice([64, 128, 256]))
        L = 2.0 * math.pi / k
        out.append((_positions(seed, n, L, amp, 1, _dtype(c), part=10 + s), L, M))
    return out


def prepare(case, seed):
    c, kind, dt = case, case["kind"], _dtype(case)
    st = {"case": c, "kind": kind}
    if kind == "batch":
        sets = _batch_sets(c, seed)
        st["batch"] = kde.Batch([s[0] for s in sets], [s[1] for s in sets], [s[2] for s in sets],
                                _log_list(1.0, 1e4, c["B"]))
        return st
    if kind == "session":
        L = c["L"]
        x = _positions(seed, c["n"], L, c["amp"], 1, dt)
        v = (c["v_th"] * torch.randn(c["n"], dtype=F64, device=DEV, generator=_rng(seed, 1))).to(dt)
        st["session"] = kde.Session(x, v, L, c["M"], c["dt"], _log_list(1.0, 1e4, c["B"]), c["n_cv"])
        return st
    L = _period(c)
    x = _positions(seed, c["n"], L, c["amp"], c["mode"], dt)
    st.update(x=x, L=L, ws=kde.Workspace(DEV))
    if kind == "scan" or kind == "refine":
        st["kappas"] = _log_list(c["k_lo"], c["k_hi"], c["B"])
    elif kind == "tri_scan":
        st["widths"] = _log_list(0.25 * L / c["M"], 0.5 * L, c["B"])
    elif kind in ("deposit", "gather"):
        st["shape"] = kde.KDE_SHAPE_TRIANGLE if c["shape"] == "tri" else kde.KDE_SHAPE_VONMISES
        st["kappa"] = _half_width(c, L) if c["shape"] == "tri" else c["kappa"]
        st["kappa_i"] = _per_particle(c, x, L) if c["per"] else None
        if kind == "gather":
            st["field"] = _field(seed, c["M"], L)
    elif kind == "widths":
        g = torch.arange(c["M"], dtype=F64, device=DEV) * (L / c["M"])
        st["pilot"] = _density(g, L, 0.9 * c["amp"], c["mode"]).contiguous()
    return st


# ---------------------------------------------------------------- one pass

def run(state):
    c, kind = state["case"], state["kind"]
    if kind == "scan":
        cv, sums, am = kde.cv_scan(state["x"], state["L"], state["kappas"], ws=state["ws"])
        return {"cv": cv, "sums": sums, "argmin": am}
    if kind == "tri_scan":
        cv, sums, am = kde.cv_scan(state["x"], state["L"], state["widths"], ws=state["ws"],
                                   shape=kde.KDE_SHAPE_TRIANGLE)
        return {"cv": cv, "sums": sums, "argmin": am}
    if kind == "refine":
        res, cv, am = kde.cv_refine(state["x"], state["L"], state["kappas"], ws=state["ws"])
        return {"result": res, "cv": cv, "argmin": am}
    if kind == "deposit":
        return {"rho": kde.deposit(state["x"], state["L"], c["M"], kappa=state["kappa"], kappa_i=state["kappa_i"],
                                   ws=state["ws"], shape=state["shape"])}
    if kind == "gather":
        return {"out": kde.gather(state["x"], state["L"], state["field"], kappa=state["kappa"],
                                  kappa_i=state["kappa_i"], shape=state["shape"])}
    if kind == "widths":
        k_i, lg, nf = kde.adapt_widths(state["x"], state["L"], state["pilot"], c["kappa"], 0.5, ws=state["ws"])
        return {"kappa_i": k_i, "log_geomean": lg, "floored": nf}
    if kind == "widths_exact":
        k_i, lg, nf = kde.adapt_widths_exact(state["x"], state["L"], c["kappa"], 0.5, ws=state["ws"])
        return {"kappa_i": k_i, "log_geomean": lg, "floored": nf}
    if kind == "batch":
        b = state["batch"]
        b.run()
        return {"kappa_star": b.kappa_star, "cv": torch.cat(b.cv), "pilot": torch.cat(b.pilot),
                "rho": torch.cat(b.rho), "kappa_i": torch.cat(b.kappa_i)}
    s = state["session"]
    s.step(c["steps"])
    return {"x": s.read(kde.KDE_SESSION_X), "v": s.read(kde.KDE_SESSION_V), "kappa": s.read(kde.KDE_SESSION_KAPPA),
            "rho": s.read(kde.KDE_SESSION_RHO), "E": s.read(kde.KDE_SESSION_E)}


# ------------------------------------------- what a pass cannot do without

def _size(c):
    return 8 if c["dtype"] == "f64" else 4


def _order(kappa):
    """About where the Fourier series of a kernel of this concentration ends."""
    return 9.0 * math.sqrt(kappa) + 8.0


def _mean_n(c):
    return (c["n_hi"] - c["n_lo"]) / math.log(c["n_hi"] / c["n_lo"])


def work(case):
    c, kind, e = case, case["kind"], _size(case)
    if kind in ("scan", "refine"):
        # moments of every particle to the series' end: a rotation and an addition each
        return {"bytes": e * c["n"] + 24 * c["B"], "flops": 8.0 * c["n"] * _order(c["k_hi"])}
    if kind == "tri_scan":
        # per particle and width, the ends of two supports and a cubic of the moments between them
        return {"bytes": e * c["n"] + 24 * c["B"], "flops": 32.0 * c["n"] * c["B"]}
    if kind in ("deposit", "gather"):
        per = e if c["per"] else 0
        out = 8 * c["M"] if kind == "deposit" else e * c["n"] + 8 * c["M"]
        if c["shape"] == "tri":
            evals = c["n"] * (2.0 * _half_width(c, _period(c)) / _period(c)) * c["M"] * 4.0
        elif c["per"]:
            evals = c["n"] * c["M"] * 8.0
        else:
            evals = c["n"] * min(8.0 * c["M"], 8.0 * _order(c["kappa"]))
        return {"bytes": (e + per) * c["n"] + out, "flops": evals}
    if kind == "widths":
        return {"bytes": 2 * e * c["n"] + 8 * c["M"], "flops": 40.0 * c["n"]}
    if kind == "widths_exact":
        return {"bytes": 2 * e * c["n"], "flops": 16.0 * c["n"] * _order(c["kappa"])}
    if kind == "batch":
        n = c["sets"] * _mean_n(c)
        return {"bytes": 2.0 * e * n, "flops": n * (8.0 * _order(1e4) + 150 * 16.0)}
    n = c["n"] * c["steps"]
    return {"bytes": 8.0 * e * n, "flops": n * c["M"] * 24.0}


# ------------------------------------------------------- the values, 64 bits

def _sin2(a, b, L):
    return torch.sin((math.pi / L) * (a - b)) ** 2


def _vm_scan(x, L, kappas):
    x = x.to(F64)
    n, B = x.shape[0], len(kappas)
    S1 = torch.zeros(B, dtype=F64, device=DEV)
    S2 = torch.zeros(B, dtype=F64, device=DEV)
    i0e = torch.special.i0e
    for lo in range(0, n, 512):
        xi = x[lo:lo + 512]
        d = xi[:, None] - x[None, lo:]
        keep = torch.ones_like(d, dtype=torch.bool).triu(1)
        phi = (math.pi / L) * d
        s2 = torch.where(keep, torch.sin(phi) ** 2, torch.full_like(d, math.inf))
        c = torch.cos(phi).abs()
        q = torch.where(keep, s2 / (1.0 + c), torch.full_like(d, math.inf))
        for b, k in enumerate(kappas):
            S2[b] += torch.exp(-2.0 * k * s2).sum()
            S1[b] += (torch.exp(-2.0 * k * q) * i0e(2.0 * k * c)).sum()
    kt = torch.tensor(np.asarray(kappas), dtype=F64, device=DEV)
    ik = i0e(kt)
    kbar0 = i0e(2.0 * kt) / (L * ik * ik)
    S1, S2 = S1 / (L * ik * ik), S2 / (L * ik)
    cv = (n * kbar0 + 2.0 * S1) / (float(n) * n) - 4.0 * S2 / (float(n) * (n - 1.0))
    return cv, torch.cat([S1, S2])


def _tri_scan(x, L, widths):
    x = x.to(F64)
    n, B = x.shape[0], len(widths)
    S1 = torch.zeros(B, dtype=F64, device=DEV)
    S2 = torch.zeros(B, dtype=F64, device=DEV)

    def spline(u):
        return ((2.0 - u).clamp(min=0.0) ** 3 - 4.0 * (1.0 - u).clamp(min=0.0) ** 3) / 6.0

    for lo in range(0, n, 512):
        xi = x[lo:lo + 512]
        d = (xi[:, None] - x[None, lo:]).abs()
        keep = torch.ones_like(d, dtype=torch.bool).triu(1)
        r = torch.where(keep, torch.minimum(d, L - d), torch.full_like(d, math.inf))
        image = torch.where(keep, L - r, torch.full_like(d, math.inf))
        for b, h in enumerate(widths):
            S2[b] += (1.0 - r / h).clamp(min=0.0).sum()
            S1[b] += spline(r / h).sum()
            if h > 0.25 * L:
                S1[b] += spline(image / h).sum()
    h = torch.tensor(np.asarray(widths), dtype=F64, device=DEV)
    S1, S2 = S1 / h, S2 / h
    cv = (n * (2.0 / (3.0 * h)) + 2.0 * S1) / (float(n) * n) - 4.0 * S2 / (float(n) * (n - 1.0))
    return cv, torch.cat([S1, S2])


def _kernel(shape, d, k, L):
    """The kernel at separations d (any image), concentrations or half-widths k."""
    if shape == "tri":
        d = d.abs()
        return (1.0 - torch.minimum(d, L - d) / k).clamp(min=0.0) / k
    return torch.exp(-2.0 * k * torch.sin((math.pi / L) * d) ** 2) / (L * torch.special.i0e(k))


def _deposit(x, k, M, L, shape="vm"):
    x, k = x.to(F64), k.to(F64)
    g = torch.arange(M, dtype=F64, device=DEV) * (L / M)
    rho = torch.zeros(M, dtype=F64, device=DEV)
    for lo in range(0, x.shape[0], 65536):
        rho += _kernel(shape, g[:, None] - x[None, lo:lo + 65536], k[None, lo:lo + 65536], L).sum(1)
    return rho / x.shape[0]


def _widths(x, f, kappa, alpha=0.5):
    lf = torch.log(f)
    lg = lf.mean()
    return (kappa * torch.exp(2.0 * alpha * (lf - lg))).to(x.dtype), lg.reshape(1)


def _interpolated(x, pilot, L):
    M = pilot.shape[0]
    u = x.to(F64) * (M / L)
    j = torch.floor(u).to(torch.int64).clamp(0, M - 1)
    t = u - j
    return (1.0 - t) * pilot[j] + t * pilot[(j + 1) % M]


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "session":
        return None
    if kind == "batch":
        kappas = _log_list(1.0, 1e4, c["B"])
        out = {"kappa_star": [], "cv": [], "pilot": [], "rho": [], "kappa_i": []}
        for x, L, M in _batch_sets(c, seed):
            cv, _ = _vm_scan(x, L, kappas)
            ks = float(kappas[int(torch.argmin(cv))])
            pilot = _deposit(x, torch.full((x.shape[0],), ks, dtype=F64, device=DEV), M, L)
            k_i, _ = _widths(x, _interpolated(x, pilot, L), ks)
            for name, v in (("kappa_star", torch.tensor([ks], dtype=F64, device=DEV)), ("cv", cv), ("pilot", pilot),
                            ("rho", _deposit(x, k_i, M, L)), ("kappa_i", k_i.to(F64))):
                out[name].append(v)
        return {name: torch.cat(v) for name, v in out.items()}
    s = prepare(case, seed)
    x, L = s["x"], s["L"]
    if kind == "scan":
        cv, sums = _vm_scan(x, L, s["kappas"])
        return {"cv": cv, "sums": sums, "argmin": None}
    if kind == "refine":
        if c["n"] > 70000:
            return None
        cv, _ = _vm_scan(x, L, s["kappas"])
        return {"result": None, "cv": cv, "argmin": None}
    if kind == "tri_scan":
        cv, sums = _tri_scan(x, L, s["widths"])
        return {"cv": cv, "sums": sums, "argmin": None}
    if kind in ("deposit", "gather"):
        k = s["kappa_i"].to(F64) if c["per"] else torch.full((c["n"],), s["kappa"], dtype=F64, device=DEV)
        if kind == "deposit":
            return {"rho": _deposit(x, k, c["M"], L, c["shape"])}
        g = torch.arange(c["M"], dtype=F64, device=DEV) * (L / c["M"])
        xd = x.to(F64)
        out = torch.empty(c["n"], dtype=F64, device=DEV)
        for lo in range(0, c["n"], 65536):
            w = _kernel(c["shape"], g[None, :] - xd[lo:lo + 65536, None], k[lo:lo + 65536, None], L)
            out[lo:lo + 65536] = (L / c["M"]) * (w * s["field"][None, :]).sum(1)
        return {"out": out}
    if kind == "widths":
        f = _interpolated(x, s["pilot"], L)
        lf = torch.log(f)
        lg = lf.mean()
        return {"kappa_i": c["kappa"] * torch.exp(lf - lg), "log_geomean": lg.reshape(1), "floored": None}
    # the exact pilot: the kernel's Fourier series with the coefficients I_m / I_0 from their backward recurrence
    xd = x.to(F64)
    order = int(10.0 * math.sqrt(c["kappa"]) + 60)
    r, ratio = 0.0, [0.0] * (order + 1)
    for m in range(order + 80, 0, -1):
        r = c["kappa"] / (2.0 * m + c["kappa"] * r)
        if m <= order:
            ratio[m] = r
    theta = (2.0 * math.pi / L) * xd
    f = torch.ones_like(xd)
    p = 1.0
    for m in range(1, order + 1):
        p *= ratio[m]
        cm, sm = torch.cos(m * theta), torch.sin(m * theta)
        f += 2.0 * p * (cm.mean() * cm + sm.mean() * sm)
    lf = torch.log(f / L)
    lg = lf.mean()
    return {"kappa_i": c["kappa"] * torch.exp(lf - lg), "log_geomean": lg.reshape(1), "floored": None}
