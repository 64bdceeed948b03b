"""The cell-wave list build with more waves than home cells, which share a cell's
atoms, against the oracle, list by list in order: parts of a cell's atoms that come
out uneven or empty, cells of more than 64 atoms, waves left over, and the
automatic choice at one, two and three tiles per CU."""
import pytest

from gpu_helpers import WCA, check_cells, check_nl, pair, state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

CASES = {
    # name: (n, rho, r_cut, reorder, nl_block, tile (x, y, z), cells per side)
    "one_cell_automatic": (4000, 0.8442, 2.5, True, 0, (0, 0, 0), 5),
    "two_cells_automatic": (10007, 0.8442, 2.5, True, 0, (0, 0, 0), 8),
    "five_cells_automatic": (50000, 0.8442, 2.5, False, 0, (5, 1, 1), 13),
    "sixteen_parts": (4000, 0.8442, 2.5, False, 1024, (1, 1, 1), 5),
    "waves_left_over": (10007, 0.8442, 2.5, True, 448, (3, 1, 1), 8),
    "more_parts_than_atoms": (4000, 0.8, WCA, True, 1024, (1, 1, 1), 12),
    "more_than_a_wave_of_homes": (11500, 3.8, 2.5, True, 192, (1, 1, 1), 5),
    "four_cells_per_side": (1500, 0.8442, 2.5, True, 512, (1, 1, 1), 4),
}


@pytest.mark.parametrize("lattice", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_lists(name, lattice):
    n, rho, rc, reorder, block, tile, nc = CASES[name]
    L, pos, vel = state(n, rho, 83, jitter=0.05 if lattice else 0.0, lattice=lattice)
    sim, s = pair(pos, vel, L, r_cut=rc, reorder=reorder)
    assert sim.grid.nc == nc
    sim.set_tuning(nl_method=md.MD_NL_CELL_WAVES, nl_block=block, tile_cells=tile[0],
                   tile_y=tile[1], tile_z=tile[2])
    sim.build_cells()
    _, cells = check_cells(sim, s, pos)
    sim.build_neighbors()
    cnt, _ = check_nl(sim, s, pos, cells)
    obs = sim.reduce()
    assert obs["flags"] == 0 and obs["max_nl"] == cnt.max()
