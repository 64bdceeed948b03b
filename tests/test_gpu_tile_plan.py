"""The tile shape chosen by itself, at its edges: grids of 3 to 5 cells per side, one
tile or several rounds of workgroups, workgroups of 64 to 1024 threads, more atoms
in a cell than fit.  Whatever the shape, the list entries keep their order, so
forces are those of tiles of one cell, bit for bit."""
import math

import numpy as np
import pytest

from gpu_helpers import WCA, pair, state

pytestmark = pytest.mark.gpu

CASES = {
    # name: (n, rho, r_cut, force_block, force_lanes, cells per side)
    "three_cells": (700, 0.8442, 2.5, 512, 2, 3),
    "four_cells": (1500, 0.8442, 2.5, 512, 2, 4),
    "five_cells": (500, 0.8, WCA, 512, 2, 6),
    "sparse": (300, 0.01, WCA, 512, 2, 21),
    "several_rounds": (32000, 0.8, WCA, 1024, 8, 24),
    "narrow_workgroups": (10007, 0.8442, 2.5, 64, 1, 8),
    "crowded_cells": (6000, 40.0, WCA, 512, 2, 3),
}


@pytest.mark.parametrize("name", list(CASES))
def test_automatic_tiles_leave_the_forces_as_they_are(name):
    n, rho, rc, block, lanes, nc = CASES[name]
    L, pos, vel = state(n, rho, 31, jitter=0.02)
    f = []
    for tile in (0, 1):
        sim, _ = pair(pos, vel, L, r_cut=rc, nl_capacity=n if rho > 2.0 else 0)
        assert sim.grid.nc == nc
        sim.set_tuning(force_block=block, force_lanes=lanes, tile_cells=tile, tile_y=tile,
                       tile_z=tile)
        sim.prepare()
        t = sim.get_tuning()
        k = [t["tile_cells"], t["tile_y"], t["tile_z"]]
        assert nc >= k[0] >= k[1] >= k[2] >= 1
        if tile == 1:
            assert k == [1, 1, 1]
        elif rho <= 2.0:
            # the expected staged atoms leave room for three workgroups per CU
            staged = math.prod(m + 2 for m in k) * n / nc ** 3
            assert (1.15 * staged + 64) * 24 <= 160 * 1024 / 3
        assert sim.reduce()["flags"] == 0
        f.append(sim.state()["f"])
    assert np.array_equal(f[0], f[1])
