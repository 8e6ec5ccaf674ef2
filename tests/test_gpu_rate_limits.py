"""Rate parameters far beyond the physical range: a reaction that a huge activation energy switches off.

Its rate constant is exp of a number below -1e3 at any temperature, that is exactly 0 in FP64: source term and
Jacobian are 0 to the last bit, not the overflow of an exponential's polynomial outside its range.
"""
import numpy as np
import pytest
import torch

from . import mechs_for_tests as mt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("rev", [1, 0])
@pytest.mark.parametrize("Ea", [1e12, 1e30, 1e60, 1e300])
def test_switched_off(tmp_path, kind, rev, Ea):
    from paper_1608_05794_amd import ck
    low = (1.0e3, 0.0, Ea) if kind >= 2 else None
    troe = (0.6, 100.0, 1000.0, 5000.0) if kind == 3 else None
    m = mt.isomer_mechanism(kind, Ea=Ea, low=low, troe=troe)
    m.reactions[0].rev = rev
    g = ck.Mechanism(mt.write(m, tmp_path / "m.ckm"))
    y, P = mt.isomer_state()
    yd, Pd = torch.as_tensor(y, device="cuda"), torch.as_tensor(P, device="cuda")
    for kernel in ("wave", "lane"):
        f, J = ck.rhs(g, yd, Pd, kernel=kernel), ck.jac(g, yd, Pd, kernel=kernel)
        print(f"[switched off] kind {kind} rev {rev} Ea {Ea:g} {kernel}: {f.abs().max().item()} {J.abs().max().item()}", flush=True)
        assert bool((f == 0.0).all()) and bool((J == 0.0).all())
    r = ck.integrate(g, yd, Pd, 1e-3)
    torch.cuda.synchronize()
    assert r["status"].item() == 0 and np.array_equal(r["y"].cpu().numpy(), y)
