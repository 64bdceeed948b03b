"""The cell offsets scanned in chunks of 4096 cells by several workgroups:
cells, lists (bit-exact) and a run across rebuilds against the oracle at grids
on both sides of one chunk, at whole chunks and at many, with more cells than
atoms and the other way round."""
import numpy as np
import pytest

import oracle
from gpu_helpers import WCA, check_cells, check_nl, min_image, pair, state

pytestmark = pytest.mark.gpu

# cells per side: one chunk exactly, one cell row past it, 2 chunks exactly short of 3, 8
# chunks, 27 chunks with mostly empty cells
CASES = {16: 18000, 17: 18000, 20: 18000, 32: 18000, 48: 17000}


@pytest.mark.parametrize("reorder", [True, False])
@pytest.mark.parametrize("nc", list(CASES))
def test_cells_and_lists(nc, reorder):
    n = CASES[nc]
    rho = n / ((nc + 0.5) * (WCA + 0.3)) ** 3
    L, pos, vel = state(n, rho, 53, lattice=False)
    sim, s = pair(pos, vel, L, r_cut=WCA, reorder=reorder)
    assert sim.grid.nc == nc
    for _ in range(2):  # the second build starts from the counts the first one left
        sim.build_cells()
        _, cells = check_cells(sim, s, pos)
    sim.build_neighbors()
    check_nl(sim, s, pos, cells)
    obs = sim.reduce()
    assert obs["max_occupancy"] == np.diff(cells[1]).max()


@pytest.mark.parametrize("nc", [17, 32])
def test_a_run_follows_the_oracle(nc):
    n = CASES[nc]
    rho = n / ((nc + 0.5) * (WCA + 0.3)) ** 3
    L, pos, vel = state(n, rho, 59, jitter=0.02)
    sim, s = pair(pos, vel, L, r_cut=WCA)
    sim.prepare()
    sim.step(30, record_every=1)
    h = sim.history()
    p_ref, v_ref, _, o_ref, nreb = oracle.run(s, pos, vel, 30)
    assert sim.reduce()["n_rebuilds"] == nreb > 0
    assert np.array_equal(h["rebuilt"], o_ref["rebuilt"])
    st = sim.state()
    assert np.abs(min_image(st["pos"] - p_ref, L)).max() < 1e-10
    assert np.abs(st["vel"] - v_ref).max() < 1e-9
