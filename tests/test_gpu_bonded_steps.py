"""Bonded systems: each reach of the terms along the chain (bonds, angles,
dihedrals) against the oracle at the parity tests' bound, and steps whose
cell sort carries the map of slots and the copy-back with it (small systems in one
workgroup, larger ones with the finish in the binning) against the same steps
without reorder, which take neither: the lists keep their order, so the
trajectories agree bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2003_14061_amd import md
from test_gpu_bonded import ALL, errors, melt, oracle_forces

pytestmark = pytest.mark.gpu

FENE = dict(fene_k=30.0, fene_r0=1.5)
TERMS = {
    "bonds": FENE,
    "bonds_angles": dict(FENE, bend_k=1.5),
    "angles": dict(bend_k=1.5),
    "dihedrals": dict(tors_c=ALL["tors_c"]),
}


@pytest.mark.parametrize("chain", [2, 4, 16])
@pytest.mark.parametrize("name", list(TERMS))
def test_each_reach_matches_the_oracle(name, chain):
    m = melt(n_side=16, M=chain)
    sim = md.Simulation(m.pos, m.vel, m.L, r_cut=m.r_cut, skin=m.skin, dt=m.dt,
                        bonded=dict(chain_length=chain, **TERMS[name]))
    sim.prepare()
    s = oracle.make_sys(m.n, m.L, r_cut=m.r_cut, skin=m.skin, dt=m.dt,
                        nl_cap=sim.grid.nl_capacity)
    ref = oracle_forces(s, oracle.make_bonded(chain, **TERMS[name]), m.pos, "tiled")
    per_atom, normwise = errors(sim.state()["f"], ref)
    assert per_atom <= 1e-12 and normwise <= 1e-12, (per_atom, normwise)
    obs = sim.reduce()
    assert obs["flags"] == 0
    assert abs(obs["U"] - ref["u"].sum()) <= 1e-12 * np.abs(ref["u"]).sum()


@pytest.mark.parametrize("n_side,every", [(16, 1), (27, 10), (32, 0)])
@pytest.mark.parametrize("graph", [False, True])
def test_steps_with_and_without_reorder(n_side, every, graph):
    m = melt(n_side=n_side, M=n_side)
    out = []
    for reorder in (True, False):
        sim = md.Simulation(m.pos, m.vel, m.L, r_cut=m.r_cut, skin=0.1, dt=0.002,
                            reorder=reorder, bonded=dict(chain_length=n_side, **ALL))
        sim.set_graph(graph)
        sim.prepare()
        for steps in (25, 16):
            sim.step(steps, record_every=every)
        obs = sim.reduce()
        assert obs["flags"] == 0
        st = sim.state()
        out.append((st["pos"], st["vel"], st["f"], obs["n_rebuilds"], obs["max_nl"]))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert out[0][3] > 3
