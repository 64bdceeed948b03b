"""Tiles of very many home rows, up to the 64 that a wave numbers, and requests past
them (reduced to 64): lists bit for bit and forces to 1e-12 against the oracle, in the
kernels that take the tiles' tables."""
import numpy as np
import pytest

import oracle
from gpu_helpers import WCA, check_cells, check_nl, force_errors, pair, state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", [md.MD_NL_LANES, md.MD_NL_CELL_WAVES])
@pytest.mark.parametrize("tile", [(2, 8, 8), (2, 9, 9), (1, 15, 4), (1, 4, 15), (1, 1000, 1000)])
@pytest.mark.parametrize("newton3", [False, True])
def test_lists_and_forces(newton3, tile, method):
    L, pos, vel = state(8788, 0.8, 109, jitter=0.05)
    sim, s = pair(pos, vel, L, r_cut=WCA, newton3=newton3)
    assert sim.grid.nc == 15
    sim.set_tuning(tile_cells=tile[0], tile_y=tile[1], tile_z=tile[2], nl_method=method)
    t = sim.get_tuning()
    assert t["tile_y"] * t["tile_z"] <= 64
    sim.build_cells()
    _, cells = check_cells(sim, s, pos)
    sim.build_neighbors()
    check_nl(sim, s, pos, cells, half=newton3)
    sim.forces()
    cnt, nl, _ = oracle.build_nl(s, sim.grid.nc, pos, cells)
    per_atom, normwise = force_errors(sim.state()["f"], oracle.forces_nl(s, pos, cnt, nl))
    assert per_atom <= 1e-12 and normwise <= 1e-12
    assert sim.reduce()["flags"] == 0
