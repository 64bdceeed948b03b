"""md_step with the integration inside the force pass against the same steps
with a separate integration pass (which md_set_timing selects).  Each atom's
kicks and drift are the same operations on the same values, so positions,
velocities, forces, rebuild steps and the energy and virial of every record
are bitwise equal; the kinetic sums add in another order (1e-13 relative, a
thousand times the rounding of a sum of positive terms in tile order)."""
import numpy as np
import pytest

from gpu_helpers import WCA, state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

CASES = {
    "wca": dict(n=2048, rho=0.8, r_cut=WCA, dt=0.005),
    "wca_fp32": dict(n=6000, rho=0.7, r_cut=WCA, dt=0.005, precision="fp32"),
    "lj": dict(n=5324, rho=0.8442, r_cut=2.5, dt=0.004),
    "lj_four_cells": dict(n=1500, rho=0.8, r_cut=2.5, dt=0.004),
    # cells only: without and with reorder, tables in LDS and past it (16 000
    # atoms), more atoms than one workgroup sorts
    "cells": dict(n=4001, rho=0.8, r_cut=WCA, dt=0.005, neighbor_list=False),
    "cells_reorder_fp32": dict(n=2500, rho=0.7, r_cut=WCA, dt=0.005, neighbor_list=False,
                               reorder=True, precision="fp32"),
    "cells_16000": dict(n=16000, rho=0.8, r_cut=WCA, dt=0.005, neighbor_list=False),
    "cells_20000_reorder": dict(n=20000, rho=0.8, r_cut=WCA, dt=0.005, neighbor_list=False,
                                reorder=True),
    "cells_lj": dict(n=4000, rho=0.8442, r_cut=2.5, dt=0.004, neighbor_list=False, block=64),
    "lj_mass_eps": dict(n=4000, rho=0.8, r_cut=2.5, dt=0.004, eps=1.3, mass=2.0),
}


def run(sep, steps, every, graph, tuning, n, rho, **kw):
    L, pos, vel = state(n, rho, 47, jitter=0.05)
    sim = md.Simulation(pos, vel, L, skin=0.3, **kw)
    if tuning:
        sim.set_tuning(**tuning)
    sim.prepare()
    sim.set_timing(sep)
    sim.set_graph(graph)
    sim.step(steps, every)
    sim.step(steps, every)
    return sim.history(), sim.reduce(), sim.state(), sim.ids()


def same(a, b):
    (ha, oa, sa, ia), (hb, ob, sb, ib) = a, b
    assert np.array_equal(ia, ib)
    for k in ("pos", "vel", "f"):
        assert np.array_equal(sa[k], sb[k]), k
    for k in ("step", "U", "W", "dmax", "rebuilt"):
        assert np.array_equal(ha[k], hb[k]), k
    assert np.allclose(ha["K"], hb["K"], rtol=1e-13, atol=0)
    assert np.allclose(ha["P"], hb["P"], rtol=0, atol=1e-13 * np.abs(sa["vel"]).sum())
    for k in ("U", "W", "K", "step", "n_rebuilds", "flags", "dmax"):
        assert oa[k] == ob[k], k


@pytest.mark.parametrize("steps,every,graph", [(1, 1, False), (2, 1, False), (9, 0, False),
                                               (15, 4, False), (16, 1, True), (38, 3, True)])
@pytest.mark.parametrize("name", list(CASES))
def test_fused_steps_are_the_separate_ones(name, steps, every, graph):
    a = run(False, steps, every, graph, None, **CASES[name])
    b = run(True, steps, every, False, None, **CASES[name])
    same(a, b)
    assert len(a[0]) == (2 * steps // every if every else 0)


@pytest.mark.parametrize("tuning", [dict(force_lanes=1, force_block=64),
                                    dict(force_lanes=8, force_block=1024),
                                    dict(stage_cap=128), dict(tile_cells=1, tile_y=1, tile_z=1)])
def test_fused_steps_of_other_launch_shapes(tuning):
    a = run(False, 20, 2, False, tuning, **CASES["lj"])
    b = run(True, 20, 2, False, tuning, **CASES["lj"])
    same(a, b)
    assert a[1]["n_rebuilds"] > 0
