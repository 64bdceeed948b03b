"""The force pass's two ways to stage a tile against the oracle (FP64 forces
1e-12 per atom and normwise, the contract of the parity tests): the rows in
registers (at most 64 staged rows, at least 5 cells per side, atoms that fit
in LDS) and the tables in LDS (any other tile), at the edges between them and
at tiles that wrap on one side, on both, or not at all along x."""
import numpy as np
import pytest

import oracle
from gpu_helpers import WCA, check_cells, check_nl, force_errors, pair, state

pytestmark = pytest.mark.gpu

CASES = {
    # name: (n, rho, r_cut, tile (x, y, z), stage_cap, cells per side)
    "rows_64": (8788, 0.8, WCA, (6, 6, 6), 0, 15),
    "tables_72_rows": (8788, 0.8, WCA, (6, 7, 6), 0, 15),
    "one_cell_tiles": (1372, 0.8, WCA, (1, 1, 1), 0, 8),
    "five_cells_both_sides_wrap": (2500, 0.8, 2.5, (5, 1, 1), 0, 5),
    "five_cells_one_tile_wide": (2500, 0.8, 2.5, (5, 5, 5), 0, 5),
    "four_cells_per_side": (1500, 0.8, 2.5, (2, 2, 2), 0, 4),
    "uneven_parts": (4000, 0.8, WCA, (4, 3, 2), 0, 12),
    "tiles_past_their_staging": (4000, 0.8, WCA, (4, 4, 4), 256, 12),
    "empty_rows": (700, 0.05, WCA, (4, 4, 4), 0, 16),
}


@pytest.mark.parametrize("lanes", [1, 2, 8])
@pytest.mark.parametrize("name", list(CASES))
def test_forces_match_the_oracle(name, lanes):
    n, rho, rc, tile, cap, nc = CASES[name]
    L, pos, vel = state(n, rho, 29, jitter=0.05)
    sim, s = pair(pos, vel, L, r_cut=rc)
    assert sim.grid.nc == nc
    sim.set_tuning(force_lanes=lanes, tile_cells=tile[0], tile_y=tile[1], tile_z=tile[2],
                   stage_cap=cap)
    sim.build_cells()
    _, cells = check_cells(sim, s, pos)
    sim.build_neighbors()
    cnt, nl = check_nl(sim, s, pos, cells)
    sim.forces()
    ref = oracle.forces_nl(s, pos, cnt, nl)
    per_atom, normwise = force_errors(sim.state()["f"], ref)
    assert per_atom <= 1e-12 and normwise <= 1e-12, (per_atom, normwise)
    obs = sim.reduce()
    assert obs["flags"] == 0
    assert abs(obs["U"] - ref["u"].sum()) <= 1e-12 * max(np.abs(ref["u"]).sum(), 1e-300)
