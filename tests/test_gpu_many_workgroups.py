"""Sizes that take the far branches of the steps' reductions and of the cell scan:
recorded fused steps of more than 8192 workgroups, whose kinetic partials go behind
the workgroups' U and W (against separate passes, as the other fused steps), and grids
of more than 4 194 304 cells, whose scan takes several rounds per workgroup (cells
and lists against the oracle)."""
import numpy as np
import pytest

from gpu_helpers import WCA, check_cells, check_nl, pair, state
from paper_2003_14061_amd import md
from test_gpu_fused_step import run, same

pytestmark = pytest.mark.gpu

# (system, tuning, workgroups of its force pass)
STEPS = {
    "cells": (dict(n=70000, rho=0.8, r_cut=WCA, dt=0.005, neighbor_list=False, reorder=True),
              None, 70000 * 32 // 256),
    "list": (dict(n=61500, rho=0.3, r_cut=2.5, dt=0.004),
             dict(tile_cells=1, tile_y=1, tile_z=1), 21 ** 3),
}


@pytest.mark.parametrize("steps,every,graph", [(7, 1, False), (12, 4, False), (12, 5, True)])
@pytest.mark.parametrize("name", list(STEPS))
def test_recorded_fused_steps(name, steps, every, graph):
    system, tuning, workgroups = STEPS[name]
    assert workgroups > 8192 and 6 * workgroups <= system["n"]
    if tuning:
        L, pos, vel = state(system["n"], system["rho"], 47, jitter=0.05)
        sim = md.Simulation(pos, vel, L, skin=0.3, r_cut=system["r_cut"], dt=system["dt"])
        assert sim.grid.nc == 21
    a = run(False, steps, every, graph, tuning, **system)
    b = run(True, steps, every, False, tuning, **system)
    same(a, b)
    assert len(a[0]) == 2 * steps // every


@pytest.mark.parametrize("reorder", [True, False])
def test_a_scan_of_several_rounds(reorder):
    nc, n = 162, 18000
    rho = n / ((nc + 0.5) * (WCA + 0.3)) ** 3
    L, pos, vel = state(n, rho, 53, lattice=False)
    # a third of the atoms close together, so that lists are not empty
    pos[: n // 3] = 0.09 * pos[: n // 3] + 0.9 * L
    sim, s = pair(pos, vel, L, r_cut=WCA, reorder=reorder, nl_capacity=64)
    assert sim.grid.nc == nc and nc ** 3 > 1024 * 4096
    for _ in range(2):  # the second build starts from the counts the first one left
        sim.build_cells()
        _, cells = check_cells(sim, s, pos)
    sim.build_neighbors()
    cnt, _ = check_nl(sim, s, pos, cells)
    assert cnt.max() > 0
    assert sim.reduce()["max_occupancy"] == np.diff(cells[1]).max()
