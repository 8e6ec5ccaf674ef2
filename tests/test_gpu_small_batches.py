"""Calls on few reactors, which take kernels of their own, against the same call on many.

A Jacobian is evaluated with one reactor per workgroup where the rounds of eight per compute unit, which
workgroups of eight reactors take, are poorly filled, and with eight per workgroup elsewhere (N <= 16: with one
always, general reactions in another build from twelve per compute unit on; N <= 24 and 33 to 36, and general
reactions of 37 to 40 rows: with one always).  All forms run the same operations in the same order, so a
reactor's matrix is the same bits in each.  The edges: the size at which the form changes, in reactors per
compute unit, or one within a form.

Timing: one reactor's call occupies one SIMD, a call on 2048 gives every SIMD two.  The form for few
reactors evaluates the rates once and stages the matrix whole, the other evaluates them for each of its
three windows (N = 64) or two: measured 27 us against 62 us at N = 64, and 65 us when one reactor took the
form for many.  The two calls alternate, so that both see the same clocks, and 0.8 of the large call's
median is the bound.
"""
import numpy as np
import pytest
import torch

from paper_1608_05794_amd import synth

from .test_gpu_shapes import draw

pytestmark = pytest.mark.gpu


def medians(calls, rounds=25):
    """Median device time of each call, taken in turn."""
    times = [[] for _ in calls]
    for r in range(rounds + 3):
        for c, call in enumerate(calls):
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            a.record()
            call()
            b.record()
            torch.cuda.synchronize()
            if r >= 3:
                times[c].append(a.elapsed_time(b))
    return [float(np.median(t)) for t in times]


def setup(tmp_path, nsp, forms, n):
    from paper_1608_05794_amd import ck
    path = str(tmp_path / "m.ckm")
    synth.write_mechanism(draw(nsp, forms), path)
    y, P = synth.reactor_states(nsp, n, "mid", seed=nsp)
    return ck, ck.Mechanism(path), torch.as_tensor(y, device="cuda"), torch.as_tensor(P, device="cuda")


@pytest.mark.parametrize("nsp,forms,per_cu", [(15, "mixed", 12), (16, "pair", 4), (31, "pair", 4), (31, "mixed", 4),
                                              (31, "all", 16), (32, "mixed", 4), (55, "pair", 4), (56, "pair", 4),
                                              (63, "all", 4), (31, "pair", 7), (39, "pair", 6), (44, "all", 7),
                                              (47, "pair", 6), (55, "pair", 5), (56, "pair", 5), (55, "mixed", 14),
                                              (63, "all", 14)])
def test_jacobian_forms_agree(tmp_path, nsp, forms, per_cu):
    edge = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    ck, g, y, P = setup(tmp_path, nsp, forms, edge + 3)
    for reactor, p in (("cp", P), ("cv", P * 2e-5)):
        many = ck.jac(g, y, p, reactor=reactor)
        for n in (1, 9, edge):
            few = ck.jac(g, y[:, :n].contiguous(), p[:n].contiguous(), reactor=reactor)
            assert torch.isfinite(few).all() and torch.equal(few, many[:, :n])


def test_jacobian_of_one_reactor_is_quicker(tmp_path):
    ck, g, y, P = setup(tmp_path, 63, "pair", 2048)
    y1, P1 = y[:, :1].contiguous(), P[:1].contiguous()
    one, many = medians([lambda: ck.jac(g, y1, P1), lambda: ck.jac(g, y, P)])
    print(f"N = 64: one reactor {1e3 * one:.1f} us, 2048 reactors {1e3 * many:.1f} us", flush=True)
    assert one <= 0.8 * many


# sizes at the edges of the tile forms; n_gen > 0 for the mixed ones
@pytest.mark.parametrize("nsp,forms", [(64, "mixed"), (79, "mixed"), (80, "all"), (95, "mixed"), (96, "pair"), (111, "pair")])
def test_ros4_tile_forms(tmp_path, nsp, forms):
    """Two reactors per compute unit (one workgroup each) and three more (one wavefront each): both within
    the shape tests' 1e-6 of the oracle, in T and in the solver's weights, after eight fixed steps."""
    from oracle import oracle as O

    from .parity_util import state_rel_error, weighted_error
    edge = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    ck, g, y, P = setup(tmp_path, nsp, forms, edge + 3)
    om = O.Mechanism(str(tmp_path / "m.ckm"))
    k = 9
    y0, P0 = y[:, :k].cpu().numpy(), P[:k].cpu().numpy()
    for h in 10.0 ** np.arange(-8, -20, -1):
        o = om.integrate(y0, P0, 8 * h, "ros4", h_fixed=h)
        if np.all(np.isfinite(o["y"])) and np.abs(o["y"][0] - y0[0]).max() < 100.0:
            break
    for n in (k, edge, edge + 3):
        r = ck.integrate(g, y[:, :n].contiguous(), P[:n].contiguous(), 8 * h, kernel="tile", h_fixed=h)
        a = r["y"][:, :k].cpu().numpy()
        eT, ew = state_rel_error(a, o["y"])[0], weighted_error(a, o["y"])
        print(f"{nsp} {forms} x {n}: T {eT:.1e} weighted {ew:.1e}", flush=True)
        assert (r["status"][:k].cpu().numpy() == 0).all() and eT <= 1e-6 and ew <= 1e-6


@pytest.mark.parametrize("nsp,forms", [(111, "pair"), (95, "all")])
def test_ros4_of_few_reactors_is_quicker(tmp_path, nsp, forms):
    """Nine reactors against four per compute unit, one round of the one-wavefront form.  With that form for
    both the times are 0.93 of each other (measured at N = 96 and 112); with a workgroup for each of the nine
    0.63 and 0.5.  The calls alternate, bound 0.8."""
    ck, g, y, P = setup(tmp_path, nsp, forms, 4 * torch.cuda.get_device_properties(0).multi_processor_count)
    y9, P9 = y[:, :9].contiguous(), P[:9].contiguous()

    def call(y, p):
        return lambda: ck.integrate(g, y, p, 8e-14, kernel="tile", h_fixed=1e-14)

    few, many = medians([call(y9, P9), call(y, P)], 11)
    print(f"{nsp} {forms}: nine reactors {few:.3f} ms, {y.shape[1]} reactors {many:.3f} ms", flush=True)
    assert few <= 0.8 * many
