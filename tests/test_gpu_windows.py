"""Paths of the ROS4 kernels that ordinary sizes do not reach, against the oracle.

Many reactions: the later column windows of the Jacobian take the first one's rate scalars from the park slice
when three rows per block of reactions fit it, and evaluate the rates again when they do not.  The mechanisms
here have each reaction of an ordinary draw several times, with the rate shared out (the same dynamics), so
that they do not fit: 3 ceil(n / 64) rows against N' of them for one wavefront, 3 ceil(n / 256) against N' / 2
for a workgroup.

Forward differences: every padded size of the kernel, N = 8 included (also with the analytic Jacobian).

Tolerances are the parity tests': identical statuses, 1e-6 in T and in the solver's weights.
"""
import copy

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1608_05794_amd import synth

from . import test_gpu_shapes as shapes
from .parity_util import state_rel_error, weighted_error

pytestmark = pytest.mark.gpu


def load(tmp_path, mech, n):
    from paper_1608_05794_amd import ck
    path = str(tmp_path / "m.ckm")
    synth.write_mechanism(mech, path)
    y, P = synth.reactor_states(len(mech.species), n, "mid", seed=len(mech.species))
    return ck, ck.Mechanism(path), O.Mechanism(path), y, P


def compare(name, r, o, k):
    a = r["y"][:, :k].cpu().numpy()
    eT, ew = state_rel_error(a, o["y"])[0], weighted_error(a, o["y"])
    print(f"  {name}: T {eT:.1e} weighted {ew:.1e}", flush=True)
    assert np.array_equal(r["status"][:k].cpu().numpy(), o["status"]) and np.all(o["status"] == 0)
    assert eT <= 1e-6 and ew <= 1e-6


@pytest.mark.parametrize("nsp,forms,copies", [(39, "pair", 6), (39, "mixed", 6), (55, "all", 6), (71, "pair", 12),
                                              (71, "mixed", 12), (111, "pair", 10)])
def test_rate_scalars_beyond_the_park_slice(tmp_path, nsp, forms, copies):
    mech = shapes.draw(nsp, forms)
    reactions = []
    for r in mech.reactions:
        r.arr = (r.arr[0] / copies,) + tuple(r.arr[1:])
        if r.low:
            r.low = (r.low[0] / copies,) + tuple(r.low[1:])
        reactions += [copy.deepcopy(r) for _ in range(copies)]
    mech.reactions = reactions
    np_wave = (nsp + 8) // 8 * 8 if nsp < 64 else (nsp + 16) // 16 * 16
    assert 3 * ((len(reactions) + 63) // 64) > np_wave
    k = 5
    many = 2 * torch.cuda.get_device_properties(0).multi_processor_count + k
    ck, g, om, y, P = load(tmp_path, mech, many)
    print(f"[park {nsp} {forms}] {len(reactions)} reactions", flush=True)
    runs = [(k, dict(kernel="wave" if nsp < 64 else "tile", precision=p)) for p in ("fp64", "fp32_refine")]
    runs += [(k, dict(kernel="group"))]
    runs += [(k, dict(kernel="wave", reactor="cv"))] if nsp < 64 else [(many, dict(kernel="tile"))]
    for n, opts in runs:
        cv = opts.get("reactor") == "cv"
        p = P / (synth.R_GAS * y[0] * (y[1:] / om.W[:, None]).sum(0)) if cv else P
        for h in 10.0 ** np.arange(-8, -20, -1):
            o = om.integrate(y[:, :k], p[:k], 4 * h, "ros4", h_fixed=h, reactor="cv" if cv else "cp")
            if np.all(np.isfinite(o["y"])) and np.abs(o["y"][0] - y[0, :k]).max() < 100.0:
                break
        r = ck.integrate(g, torch.as_tensor(np.ascontiguousarray(y[:, :n]), device="cuda"),
                         torch.as_tensor(p[:n].copy(), device="cuda"), 4 * h, h_fixed=h, **opts)
        compare(f"{opts} x {n} h {h:.0e}", r, o, k)


@pytest.mark.parametrize("nsp,forms", [(7, "pair"), (15, "mixed"), (16, "pair"), (23, "all"), (31, "pair"), (32, "mixed"),
                                       (39, "pair"), (47, "mixed"), (48, "pair"), (55, "all"), (56, "pair"), (63, "mixed")])
@pytest.mark.parametrize("reactor", ["cp", "cv"])
def test_forward_differences(tmp_path, nsp, forms, reactor):
    k = 4
    ck, g, om, y, P = load(tmp_path, shapes.draw(nsp, forms), k)
    p = P if reactor == "cp" else P / (synth.R_GAS * y[0] * (y[1:] / om.W[:, None]).sum(0))
    # the longest of these horizons that the oracle crosses in at most 80 attempted steps a reactor
    for te in 10.0 ** np.arange(-6, -20, -1):
        o = om.integrate(y, p, te, "ros4", jacobian="fd", reactor=reactor, max_steps=80)
        if np.all(o["status"] == 0):
            break
    print(f"[fd {nsp} {forms} {reactor}] to {te:.0e} s in {o['n_accept'] + o['n_reject']}", flush=True)
    r = ck.integrate(g, torch.as_tensor(y, device="cuda"), torch.as_tensor(p, device="cuda"), te, kernel="wave",
                     jacobian="fd", reactor=reactor)
    compare("fd", r, o, k)


@pytest.mark.parametrize("forms", ["pair", "mixed", "all"])
def test_eight_rows(tmp_path, forms):
    """N = 8: every integrator of this size over eight fixed steps, the largest over which the oracle stays
    finite and T moves by less than 100 K (these seven-species draws need steps below 1e-20 s for that)."""
    k = 13
    ck, g, om, y, P = load(tmp_path, shapes.draw(7, forms), k)
    yd = torch.as_tensor(y, device="cuda")
    fo = om.rhs(y, P)
    err = np.abs(ck.rhs(g, yd, torch.as_tensor(P, device="cuda")).cpu().numpy() - fo)
    assert (err <= 1e-12 * shapes.gross_rates(shapes.draw(7, forms), om, y, P)).all()
    for method, opts in [("ros4", {}), ("ros4", dict(precision="fp32_refine")), ("ros4", dict(kernel="group")),
                         ("ros4", dict(kernel="lane")), ("rkf45", {}), ("ros4", dict(reactor="cv")),
                         ("rkf45", dict(reactor="cv"))]:
        cv = "reactor" in opts
        p = P / (synth.R_GAS * y[0] * (y[1:] / om.W[:, None]).sum(0)) if cv else P
        for h in 10.0 ** np.arange(-8, -26, -1):
            o = om.integrate(y, p, 8 * h, method, h_fixed=h, reactor="cv" if cv else "cp")
            if np.all(np.isfinite(o["y"])) and np.abs(o["y"][0] - y[0]).max() < 100.0:
                break
        r = ck.integrate(g, yd, torch.as_tensor(p, device="cuda"), 8 * h, method=method, h_fixed=h, **opts)
        compare(f"{method} {opts} h {h:.0e}", r, o, k)
