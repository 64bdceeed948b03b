"""Pairs across the periodic boundary that are in or out of the list by the last
rounding: their raw difference taken first and then the image (the inclusion
test's order), or the image first and then the difference, decide differently.
The cell-wave build (one wave per home cell and several) and the lane build, in
units from 1e-10 to 1e12 of the usual ones, against the oracle, list by list in
order."""
import numpy as np
import pytest

from gpu_helpers import WCA, check_cells, check_nl, pair
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

TUNING = {
    "waves": dict(nl_method=md.MD_NL_CELL_WAVES),
    "several_waves_per_cell": dict(nl_method=md.MD_NL_CELL_WAVES, nl_block=1024, tile_cells=2,
                                   tile_y=1, tile_z=1),
    "lanes": dict(nl_method=md.MD_NL_LANES),
}


def edge_pairs(L, rl, want, rng):
    """Coordinates (low, high) of pairs whose separation across the boundary is the
    list radius to a rounding, and the two orders disagree, from one side or the
    other."""
    rl2 = rl * rl
    out = []
    while len(out) < want:
        a = rng.uniform(0.0, 0.9 * rl)
        b = a + L - rl
        for _ in range(3):
            b = np.nextafter(b, 0.0)
        for _ in range(7):
            inside = ((a - b) + L) ** 2 < rl2
            if inside != ((a - (b - L)) ** 2 < rl2) or inside != ((b - (a + L)) ** 2 < rl2):
                out.append((a, b))
                break
            b = np.nextafter(b, L)
    return np.array(out)


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("unit", [1.0, 1e-10, 1e12])
@pytest.mark.parametrize("name", list(TUNING))
def test_pairs_at_the_list_radius(name, unit, axis):
    rng = np.random.default_rng(91)
    r_cut, skin = WCA * unit, 0.3 * unit
    L = 9.3 * (r_cut + skin)
    ab = edge_pairs(L, r_cut + skin, 300, rng)
    side = rng.uniform(0.0, L, (len(ab), 2))
    ends = [np.insert(side, axis, ab[:, e], axis=1) for e in (0, 1)]
    pos = np.concatenate(ends + [rng.uniform(0.0, L, (1500, 3))])
    assert pos.max() < L
    sim, s = pair(pos, np.zeros_like(pos), L, r_cut=r_cut, skin=skin, sigma=unit)
    assert sim.grid.nc == 9
    sim.set_tuning(**TUNING[name])
    sim.build_cells()
    _, cells = check_cells(sim, s, pos)
    sim.build_neighbors()
    check_nl(sim, s, pos, cells)
