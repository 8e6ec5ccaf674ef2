"""Calls on few reactors, which take kernels of their own, against the same call on many.

A Jacobian is evaluated with one reactor per workgroup up to four per compute unit and with eight beyond
that (N <= 16: with one always, general reactions in another build from twelve per compute unit on; general
reactions and N <= 32: with one again from sixteen on).  All forms run the same operations in the same order,
so a reactor's matrix is the same bits in each.

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
                                              (63, "all", 4)])
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
