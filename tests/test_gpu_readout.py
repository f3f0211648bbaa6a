"""Copies of results to the caller at the sizes where the way of copying
changes (one copy up to 2 MiB, the runtime's up to 48, a ring of chunks and
threads above), whole and with some outputs left out. At t = 0 the fields are
the inputs to rounding (sums of nine populations: below 1e-14), and every
value differs from its neighbours."""
import ctypes

import numpy as np
import pytest

import workloads
from paper_2109_12565_amd import Simulation

pytestmark = pytest.mark.gpu


def make(lx, ly):
    rng = np.random.default_rng(lx * 10000 + ly)
    init = {k: rng.uniform(0.3, 1.2, (ly, lx)) for k in ("rho_a", "rho_b", "temp")}
    w = workloads.small()
    return Simulation(w["params"], init["rho_a"], init["rho_b"], init["temp"], precision="fp64",
                      t_bottom=np.ones(lx)), init


# 40 bytes a node: 26214 nodes are 1 MiB; 4 MiB chunks, 2 MiB windows
@pytest.mark.parametrize("lx,ly", [(5, 3), (128, 64), (243, 215), (244, 215), (647, 648), (647, 649),
                                   (1024, 512), (1228, 1024), (1230, 1024),
                                   (1999, 1021)])
def test_fields_at_the_sizes_where_the_copy_changes(lx, ly):
    sim, init = make(lx, ly)
    with sim:
        f = sim.fields()
        for k, v in init.items():
            assert np.allclose(f[k], v, rtol=1e-13, atol=0), k
        g = sim.fields()
        assert all(np.array_equal(f[k], g[k]) for k in f)
        # two outputs left out: what is asked for comes, unaligned destinations too
        n = lx * ly
        room = np.full(3 * n + 3, -1.0)
        out = [room[1:1 + n], None, None, room[1 + n:1 + 2 * n], room[1 + 2 * n:1 + 3 * n]]
        dp = ctypes.POINTER(ctypes.c_double)
        rc = sim._lib.tlb_get_fields(sim._h, *(None if o is None else o.ctypes.data_as(dp) for o in out))
        assert rc == 0
        assert np.array_equal(out[0], f["rho_a"].ravel())
        assert np.array_equal(out[3], f["uy"].ravel())
        assert np.array_equal(out[4], f["temp"].ravel())
        assert room[0] == -1.0 and (room[1 + 3 * n:] == -1.0).all()
