"""The list build with a lane per home atom against the oracle, list by list in order:
runs of candidates below and past the 32 of a mask, empty cells, tiles that
wrap on one side and on both, grids under 5 cells per side, lists past their
capacity, and a lattice spaced by the list radius, whose pairs are in or out by
the last rounding, across the periodic boundary as inside."""
import numpy as np
import pytest

from gpu_helpers import WCA, check_cells, check_nl, pair, state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

CASES = {
    # name: (n, rho, r_cut, tile (x, y, z), cells per side)
    "sparse": (8788, 0.8, WCA, (0, 0, 0), 15),
    "empty_cells": (700, 0.05, WCA, (4, 4, 4), 16),
    "runs_past_32": (5300, 0.4822, 2.5, (2, 2, 1), 7),
    "runs_past_64": (2500, 0.8, 2.5, (1, 1, 1), 5),
    "one_tile_wide": (2500, 0.8, 2.5, (5, 1, 1), 5),
    "four_cells": (1500, 0.8, 2.5, (2, 1, 1), 4),
    "three_cells": (700, 0.8, 2.5, (1, 1, 1), 3),
}


def build(sim, s, pos):
    sim.build_cells()
    _, cells = check_cells(sim, s, pos)
    sim.build_neighbors()
    return check_nl(sim, s, pos, cells)[0]


@pytest.mark.parametrize("lattice", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_lists(name, lattice):
    n, rho, rc, tile, nc = CASES[name]
    L, pos, vel = state(n, rho, 71, jitter=0.05 if lattice else 0.0, lattice=lattice)
    sim, s = pair(pos, vel, L, r_cut=rc)
    assert sim.grid.nc == nc
    sim.set_tuning(nl_method=md.MD_NL_LANES, tile_cells=tile[0], tile_y=tile[1], tile_z=tile[2])
    cnt = build(sim, s, pos)
    obs = sim.reduce()
    assert obs["flags"] == 0 and obs["max_nl"] == cnt.max()


@pytest.mark.parametrize("shift", [0.0, 0.37, 0.93])
@pytest.mark.parametrize("m", [6, 9])
def test_pairs_at_the_list_radius(m, shift):
    rl = WCA + 0.3
    L = m * rl * (1.0 + 1e-15)
    k = (np.arange(m) + shift) * rl % L
    pos = np.stack(np.meshgrid(k, k, k, indexing="ij"), -1).reshape(-1, 3)
    pos = np.concatenate([pos, (pos + [0.5, 0.25, 0.0]) % L])
    sim, s = pair(pos, np.zeros_like(pos), L, r_cut=WCA)
    assert sim.grid.nc >= 5
    sim.set_tuning(nl_method=md.MD_NL_LANES)
    cnt = build(sim, s, pos)
    assert cnt.min() >= 1


@pytest.mark.parametrize("cap", [4, 8, 12])
def test_lists_past_the_capacity_keep_their_first_entries(cap):
    L, pos, vel = state(8788, 0.8, 73, jitter=0.05)
    full, _ = pair(pos, vel, L, r_cut=WCA)
    short, _ = pair(pos, vel, L, r_cut=WCA, nl_capacity=cap)
    for sim in (full, short):
        sim.set_tuning(nl_method=md.MD_NL_LANES)
        sim.build_cells()
        sim.build_neighbors()
    cnt, nl = full.neighbor_list()
    cnt_s, nl_s = short.neighbor_list()
    n = len(pos)
    assert np.array_equal(cnt_s[:n], np.minimum(cnt[:n], cap))
    m = np.arange(cap)[:, None] < cnt_s[None, :n]
    assert np.array_equal(np.where(m, nl_s[:, :n], -1), np.where(m, nl[:cap, :n], -1))
    obs = short.reduce(check=False)
    longest = cnt[:n].max()
    assert obs["max_nl"] == longest and bool(obs["flags"] & 1) == (longest > cap)
