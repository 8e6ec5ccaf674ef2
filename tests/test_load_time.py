"""Loading a mechanism: choosing the lanes of its pair-form reactions stays in proportion to reading the file.

The choice is made on the host for every loaded mechanism.  The same file with every reaction irreversible has
no pair-form reaction and so nothing to choose: loading it is reading and packing.  The whole load may take up
to four times that (measured: 2.4 times at 325 reactions, 2.8 at 784; 18 to 20 times while every exchange
counted whole groups of lanes anew).  Without a device the call ends with CK_EHIP after this work.
"""
import ctypes as C
import os
import time

import pytest

from paper_1608_05794_amd import synth


@pytest.mark.parametrize("name", ["M53", "M111"])
def test_lane_choice_in_proportion(tmp_path, name):
    from paper_1608_05794_amd import ck
    if not os.path.exists(ck.LIB_PATH):
        from paper_1608_05794_amd import build
        build.build()
    mech = synth.make_mechanism(name)
    paths = [str(tmp_path / "pair.ckm"), str(tmp_path / "general.ckm")]
    synth.write_mechanism(mech, paths[0])
    for r in mech.reactions:
        r.rev = 0
    synth.write_mechanism(mech, paths[1])

    def load(path):
        h = C.c_void_p()
        t0 = time.perf_counter()
        rc = ck.lib().ck_mechanism_load(path.encode(), 0, C.byref(h))
        t = time.perf_counter() - t0
        assert rc in (0, -5)
        if rc == 0:
            ck.lib().ck_mechanism_free(h)
        return t

    best = [1e9, 1e9]
    for _ in range(8):
        for i, p in enumerate(paths):
            best[i] = min(best[i], load(p))
    print(f"{name}: {1e3 * best[0]:.2f} ms, without pair-form reactions {1e3 * best[1]:.2f} ms")
    assert best[0] <= 4.0 * best[1]
