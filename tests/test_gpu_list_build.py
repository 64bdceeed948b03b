"""The cell-wave list build against the oracle, list by list in order: more
candidates than one block of registers holds (lists that cross blocks at every
chunk offset), home cells of more than 64 atoms, cells on one and on both
periodic boundaries, slots in and out of cell order, workgroups without room
for the queues, and lists past their capacity."""
import numpy as np
import pytest

from gpu_helpers import WCA, check_cells, check_nl, pair, state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

CASES = {
    # name: (n, rho, r_cut, reorder, tuning, cells per side)
    "dense_liquid": (10976, 0.8442, 2.5, True, {}, 8),
    "dense_liquid_unordered": (6912, 0.8442, 2.5, False, {}, 7),
    "several_blocks": (6600, 2.2, 2.5, True, {}, 5),
    "more_than_a_wave_of_homes": (11500, 3.8, 2.5, True, {}, 5),
    "wide_tiles": (10976, 0.8442, 2.5, True, dict(tile_cells=4, tile_y=3, tile_z=2), 8),
    "twelve_waves": (32000, 0.8442, 2.5, False, dict(tile_cells=3, tile_y=2, tile_z=2), 11),
    "no_room_for_queues": (10976, 0.8442, 2.5, True, dict(stage_cap=6600), 8),
    "tiles_past_their_staging": (10976, 0.8442, 2.5, True, dict(stage_cap=512), 8),
    "sparse_cells": (8788, 0.8, WCA, True, dict(nl_method=md.MD_NL_CELL_WAVES), 15),
    "one_wave": (10976, 0.8442, 2.5, True, dict(nl_block=64), 8),
}


@pytest.mark.parametrize("lattice", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_lists(name, lattice):
    n, rho, rc, reorder, tuning, nc = CASES[name]
    L, pos, vel = state(n, rho, 61, jitter=0.05 if lattice else 0.0, lattice=lattice)
    sim, s = pair(pos, vel, L, r_cut=rc, reorder=reorder)
    assert sim.grid.nc == nc
    if tuning:
        sim.set_tuning(**tuning)
    sim.set_tuning(nl_method=md.MD_NL_CELL_WAVES)
    sim.build_cells()
    _, cells = check_cells(sim, s, pos)
    sim.build_neighbors()
    o_cnt, _ = check_nl(sim, s, pos, cells)
    obs = sim.reduce()
    assert obs["flags"] == 0 and obs["max_nl"] == o_cnt.max()


@pytest.mark.parametrize("cap", [4, 60, 72])
def test_lists_past_the_capacity_keep_their_first_entries(cap):
    L, pos, vel = state(10976, 0.8442, 67, jitter=0.05)
    full, _ = pair(pos, vel, L, r_cut=2.5)
    short, _ = pair(pos, vel, L, r_cut=2.5, nl_capacity=cap)
    for sim in (full, short):
        sim.build_cells()
        sim.build_neighbors()
    cnt, nl = full.neighbor_list()
    cnt_s, nl_s = short.neighbor_list()
    n = len(pos)
    assert np.array_equal(cnt_s[:n], np.minimum(cnt[:n], cap))
    m = np.arange(cap)[:, None] < cnt_s[None, :n]
    assert np.array_equal(np.where(m, nl_s[:, :n], -1), np.where(m, nl[:cap, :n], -1))
    obs = short.reduce(check=False)
    assert obs["flags"] & 1 and obs["max_nl"] == cnt[:n].max()
