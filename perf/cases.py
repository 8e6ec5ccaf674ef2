"""Performance cases of the batched chemical-kinetics library.

A case is one call of the package's public entry points on device-resident reactor states: the
source term (`ck.rhs`), the analytic Jacobian (`ck.jac`), a ROS4 or RKF45 integration
(`ck.integrate`) or the graph-driven step loop (`ck.integrate_graph`).  Mechanisms are the
package's seeded synthetic ones (13, 53 and 111 species) and states its seeded recipes, the same
that the benchmark and the tests use.

Integrations run from the initial state to the case's end time.  The attempted-step counters of an
integration are not among the outputs: whether a step with an error of almost exactly 1 is accepted
is decided by rounding, so two correct summation orders may differ by a step in a million, while the
state at the end time does not move beyond the solver's tolerance.
"""
import math

import numpy as np
import torch

from paper_1608_05794_amd import ck, synth

# state recipe of each mechanism, its size, and the operations of one source term, Jacobian, ROS4
# step and RKF45 step (FMA = 2, exp / log = 20, dense LU (2/3) N^3)
MECH = {
    "M13": dict(recipe="small", nsp=13, rhs=2888, jac=5580, ros4=15285, rkf45=17888),
    "M53": dict(recipe="mid", nsp=53, rhs=30501, jac=66895, ros4=260413, rkf45=185166),
    "M111": dict(recipe="divergent", nsp=111, rhs=69567, jac=189771, ros4=1381107, rkf45=421882),
}
# mean attempted steps per reactor to an end time (log10 s), rtol 1e-8, atol 1e-12
STEPS = {
    ("M13", "ros4"): [(-12, 387), (-10, 400), (-8, 599), (-6, 1089), (-4, 1643)],
    ("M53", "ros4"): [(-14, 229), (-13, 457), (-12, 643), (-11, 886), (-10, 1269)],
    ("M111", "ros4"): [(-14, 223), (-13, 302), (-12, 477)],
    ("M13", "rkf45"): [(-14, 95), (-13, 151), (-12, 619)],
    ("M53", "rkf45"): [(-14, 54), (-13, 144)],
}
# a drawn case's operations: never more than the largest listed one's (16384 reactors of M53)
MAX_FLOPS = 0.9 * 16384 * 457 * 260413.0


def listed():
    return [
        # latency of the smallest call: the source term of one wave of reactors, as a solver's
        # right-hand-side callback makes it
        dict(name="rhs_m13_64", path="rhs", mech="M13", n=64),
        # the source-term benchmark: a full batch of the mid configuration
        dict(name="rhs_m53_131072", path="rhs", mech="M53", n=131072),
        # source term at the largest mechanism, two state components per lane, ragged batch
        dict(name="rhs_m111_30011", path="rhs", mech="M111", n=30011),
        # Jacobians handed to a caller's own implicit solver: N^2 values per reactor leave the chip
        dict(name="jac_m53_8192", path="jac", mech="M53", n=8192),
        dict(name="jac_m111_1999", path="jac", mech="M111", n=1999),
        # the small configuration as it stands: 1024 reactors to 1e-4 s
        dict(name="ros4_m13_1024", path="ros4", mech="M13", n=1024, t_end=1e-4),
        # a small request of the serving stream: latency of a chain of dependent steps
        dict(name="ros4_m53_5", path="ros4", mech="M53", n=5, t_end=1e-11),
        # the mid configuration with every resident wavefront busy and several reactors queued for each
        dict(name="ros4_m53_16384", path="ros4", mech="M53", n=16384, t_end=1e-13),
        # the precision configuration: FP32 factorisation refined in FP64
        dict(name="refined_m53_4096", path="refined", mech="M53", n=4096, t_end=1e-13),
        # the batching configuration: half hot, half cold, step counts diverge; ragged batch
        dict(name="ros4_m111_4099", path="ros4", mech="M111", n=4099, t_end=1e-13),
        # the explicit pair on the mid mechanism over a horizon that its stability bound allows
        dict(name="rkf45_m53_8191", path="rkf45", mech="M53", n=8191, t_end=1e-13),
        # the graph-driven step loop on short launches
        dict(name="graph_m13_4096", path="graph", mech="M13", n=4096, t_end=1e-8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: sizes log-uniform, end times log-uniform."""
    path = rng.choice(["rhs", "rhs", "jac", "jac", "ros4", "ros4", "ros4", "refined", "rkf45", "graph", "cv"])
    if path == "rhs":
        mech = rng.choice(["M13", "M53", "M111"])
        return dict(path=path, mech=mech, n=_log_int(rng, 1, 131072), reactor=rng.choice(["cp", "cp", "cv"]))
    if path == "jac":
        mech = rng.choice(["M13", "M53", "M111"])
        return dict(path=path, mech=mech, n=_log_int(rng, 1, {"M13": 65536, "M53": 8192, "M111": 2048}[mech]))
    mech = rng.choice(["M13", "M53", "M111"] if path in ("ros4", "refined") else
                      ["M13", "M53"] if path in ("rkf45", "cv") else ["M13"])
    method = "rkf45" if path == "rkf45" else "ros4"
    tab = STEPS[(mech, method)]
    hi = min(tab[-1][0], -8) if path == "graph" else tab[-1][0]
    lt = rng.uniform(tab[0][0], hi)
    c = dict(path=path, mech=mech, n=1, t_end=float("%.3g" % 10 ** lt))
    most = 0.25 * MAX_FLOPS / (_steps(c) * MECH[mech][method])
    # small mechanisms run below the arithmetic rate of the larger ones: fewer reactors
    cap = {"M13": 16384, "M53": 16384, "M111": 4096}[mech] // (4 if path in ("refined", "graph") else 1)
    c["n"] = _log_int(rng, 1, max(1, min(most, cap)))
    return c


def _method(case):
    return "rkf45" if case["path"] == "rkf45" else "ros4"


def _steps(case):
    tab = STEPS[(case["mech"], _method(case))]
    return float(np.interp(math.log10(case["t_end"]), [a for a, _ in tab], [b for _, b in tab]))


_handles = {}


def _mechanism(name):
    """A program loads a mechanism once and keeps its handle."""
    if name not in _handles:
        _handles[name] = ck.Mechanism(synth.mechanism_file(name))
    return _handles[name]


def _inputs(case, seed):
    """State [N, n] and pressures (densities where the case is at constant volume), on the host."""
    m = MECH[case["mech"]]
    y, p = synth.reactor_states(m["nsp"], case["n"], m["recipe"], seed=seed)
    if _reactor(case) == "cv":
        W = np.array([s.W for s in synth.make_mechanism(case["mech"]).species])
        p = p / (synth.R_GAS * y[0] * (y[1:] / W[:, None]).sum(axis=0))
    return y, p


def _reactor(case):
    return "cv" if case["path"] == "cv" or case.get("reactor") == "cv" else "cp"


def prepare(case, seed):
    y, p = _inputs(case, seed)
    return dict(case=case, mech=_mechanism(case["mech"]), y=torch.as_tensor(y, device="cuda"),
                p=torch.as_tensor(p, device="cuda"))


def run(state):
    case, mech, y, p = state["case"], state["mech"], state["y"], state["p"]
    path = case["path"]
    if path == "rhs":
        return ck.rhs(mech, y, p, reactor=_reactor(case))
    if path == "jac":
        return ck.jac(mech, y, p)
    if path == "graph":
        # eight attempted steps per launch, sixteen launches per graph: a few tenths of a
        # millisecond per launch, where the launch loop itself counts
        r = ck.integrate_graph(mech, y, p, case["t_end"], launch_steps=8, launches_per_graph=16)
    else:
        opts = {"refined": dict(precision="fp32_refine"), "cv": dict(reactor="cv")}.get(path, {})
        r = ck.integrate(mech, y, p, case["t_end"], method=_method(case), **opts)
    return dict(T=r["y"][0], Y=r["y"][1:], status=r["status"])


def work(case):
    m, n = MECH[case["mech"]], case["n"]
    N = m["nsp"] + 1
    if case["path"] == "rhs":
        return dict(bytes=8.0 * n * (2 * N + 1), flops=float(n * m["rhs"]))
    if case["path"] == "jac":
        return dict(bytes=8.0 * n * (N * N + N + 1), flops=float(n * m["jac"]))
    # state in and out, pressure, end time, status and two step counters
    return dict(bytes=n * (8.0 * (2 * N + 2) + 12), flops=n * _steps(case) * m[_method(case)])


# --- the same quantities in plain torch, 64 bits -----------------------------------------------------

_tables = {}


def _table(name, dev):
    """Parameters of a mechanism as dense tensors."""
    if (name, dev) in _tables:
        return _tables[(name, dev)]
    m = synth.make_mechanism(name)
    ns, nr = len(m.species), len(m.reactions)
    nf, nb, al = (np.zeros((nr, ns)) for _ in range(3))
    arr, low, troe = np.zeros((nr, 3)), np.zeros((nr, 3)), np.ones((nr, 4))
    typ, rev = np.zeros(nr, dtype=np.int64), np.zeros(nr)
    low[:, 0] = 1.0
    for i, r in enumerate(m.reactions):
        for k, v in r.reac:
            nf[i, k] += v
        for k, v in r.prod:
            nb[i, k] += v
        arr[i], typ[i], rev[i] = r.arr, r.type, r.rev
        if r.type:
            al[i] = 1.0
            for k, a in r.eff:
                al[i, k] = a
        if r.type >= 2:
            low[i] = r.low
        if r.type == 3:
            troe[i] = r.troe
    t = dict(W=np.array([s.W for s in m.species]), lo=np.array([s.a_low for s in m.species]),
             hi=np.array([s.a_high for s in m.species]), nf=nf, nb=nb, al=al, arr=arr, low=low, troe=troe,
             typ=typ, rev=rev, ff=_factors(nf, ns), fb=_factors(nb, ns))
    _tables[(name, dev)] = {k: torch.as_tensor(v, device=dev) for k, v in t.items()}
    return _tables[(name, dev)]


def _factors(nu, ns):
    """Species of each reaction's mass-action product, one column per factor (ns: the factor 1)."""
    out = np.full((nu.shape[0], int(nu.sum(axis=1).max())), ns)
    for i, row in enumerate(nu.astype(int)):
        f = [k for k, v in enumerate(row) for _ in range(v)]
        out[i, :len(f)] = f
    return out


def _power_products(C, factors):
    """prod_k C_k^nu_ik (reactions x reactors)."""
    C1 = torch.cat([C, torch.ones_like(C[:1])])
    out = C1[factors[:, 0]]
    for c in range(1, factors.shape[1]):
        out = out * C1[factors[:, c]]
    return out


def _plain_rhs(m, y, p, cv):
    R, p0 = synth.R_GAS, synth.P0
    T, Y = y[0], y[1:]
    S = (Y / m["W"][:, None]).sum(0)
    rho = p if cv else p / (R * T * S)
    C = rho * Y / m["W"][:, None]
    a = torch.where((T < synth.T_MID)[None, :, None], m["lo"][:, None, :], m["hi"][:, None, :])
    cp = a[..., 0] + T * (a[..., 1] + T * (a[..., 2] + T * (a[..., 3] + T * a[..., 4])))
    H = a[..., 0] + T * (a[..., 1] / 2 + T * (a[..., 2] / 3 + T * (a[..., 3] / 4 + T * a[..., 4] / 5))) + a[..., 5] / T
    Sr = a[..., 0] * torch.log(T) + T * (a[..., 1] + T * (a[..., 2] / 2 + T * (a[..., 3] / 3 + T * a[..., 4] / 4))) \
        + a[..., 6]
    nu = m["nb"] - m["nf"]
    lnT = torch.log(T)
    lnk = torch.log(m["arr"][:, :1]) + m["arr"][:, 1:2] * lnT - m["arr"][:, 2:] / (R * T)
    lnK = -nu @ (H - Sr) + nu.sum(1)[:, None] * torch.log(p0 / (R * T))
    kf, kr = torch.exp(lnk), m["rev"][:, None] * torch.exp(lnk - lnK)
    Mc = m["al"] @ C
    lnk0 = torch.log(m["low"][:, :1]) + m["low"][:, 1:2] * lnT - m["low"][:, 2:] / (R * T)
    Pr = torch.exp(lnk0 - lnk) * Mc
    A, T3, T1, T2 = (m["troe"][:, i:i + 1] for i in range(4))
    Fc = (1 - A) * torch.exp(-T / T3) + A * torch.exp(-T / T1) + torch.exp(-T2 / T)
    typ = m["typ"][:, None]
    # reactions without fall-off carry harmless values through these lines
    LF = torch.log10(torch.where(typ == 3, Fc, torch.ones_like(Fc)).clamp_min(1e-300))
    c0, n0 = -0.4 - 0.67 * LF, 0.75 - 1.27 * LF
    x = torch.log10(torch.where(typ >= 2, Pr, torch.ones_like(Pr)).clamp_min(1e-300)) + c0
    F = torch.pow(10.0, LF / (1 + (x / (n0 - 0.14 * x)) ** 2))
    fall = Pr / (1 + Pr) * torch.where(typ == 3, F, torch.ones_like(F))
    c = torch.where(typ == 0, torch.ones_like(Mc), torch.where(typ == 1, Mc, fall))
    q = c * (kf * _power_products(C, m["ff"]) - kr * _power_products(C, m["fb"]))
    wd = nu.T @ q
    if cv:
        Q, cap = R * T * ((H - 1) * wd).sum(0), R * (Y * (cp - 1) / m["W"][:, None]).sum(0)
    else:
        Q, cap = R * T * (H * wd).sum(0), R * (Y * cp / m["W"][:, None]).sum(0)
    return torch.cat([(-Q / (rho * cap))[None], m["W"][:, None] * wd / rho])


def exact(case, seed):
    if case["path"] not in ("rhs", "jac"):
        return None     # a stiff integration to far tighter tolerances takes minutes
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    m = _table(case["mech"], dev)
    y, p = (torch.as_tensor(v, device=dev) for v in _inputs(case, seed))
    cv = _reactor(case) == "cv"
    N, n = y.shape
    if case["path"] == "rhs":
        return torch.cat([_plain_rhs(m, y[:, i:i + 16384], p[i:i + 16384], cv) for i in range(0, n, 16384)], dim=1)
    J = torch.empty((N, N, n), dtype=torch.float64, device=dev)
    for i in range(0, n, 8192):
        yi, pi = y[:, i:i + 8192].contiguous(), p[i:i + 8192]
        for j in range(N):
            e = torch.zeros_like(yi)
            e[j] = 1.0
            J[:, j, i:i + 8192] = torch.func.jvp(lambda v: _plain_rhs(m, v, pi, cv), (yi,), (e,))[1]
    return J.reshape(N * N, n)
