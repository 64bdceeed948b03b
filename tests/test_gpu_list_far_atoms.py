"""Atoms that left the box by several box lengths in one step (a blow-up elsewhere, or
an absurd velocity): folded by one length only, they stay in the cells at the box's
edges among ordinary atoms, whose lists have to be whole.  The cell-wave build, which
prunes candidates by the box of a cell's atoms, against the lane build, which tests
every pair by itself, list by list in order."""
import numpy as np
import pytest

from gpu_helpers import state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

FAR = [-3.3, -1.6, 2.2, 7.0, 40.0, -1e4, 1e9, -1e9]


def lists(sim, method, **kw):
    sim.set_tuning(nl_method=method, **kw)
    sim.build_cells()
    sim.build_neighbors()
    cnt, nl = sim.neighbor_list()
    n, ids = sim.n, sim.ids()
    m = np.arange(nl.shape[0])[:, None] < cnt[None, :n]
    by_id = np.empty((n, nl.shape[0]), np.int64)
    by_id[ids] = np.where(m, ids[np.clip(nl[:, :n], 0, n - 1)], -1).T
    return by_id


@pytest.mark.parametrize("nl_block", [0, 1024])
@pytest.mark.parametrize("reorder", [True, False])
@pytest.mark.parametrize("far", [FAR, [1.3, -1.2], [-1.7], [-1e9]])
def test_lists_beside_atoms_far_outside(far, reorder, nl_block):
    L, pos, vel = state(4000, 0.8442, 113, jitter=0.05)
    dt = 0.004
    rng = np.random.default_rng(7)
    for k, i in enumerate(rng.choice(len(pos), 3 * len(far), replace=False)):
        vel[i, k % 3] = far[k // 3] * L / dt
    sims = [md.Simulation(pos, vel, L, r_cut=2.5, dt=dt, skin=0.3, reorder=reorder,
                          nl_capacity=400) for _ in range(2)]
    for sim in sims:
        sim.set_tuning(nl_method=md.MD_NL_LANES)
        sim.prepare()
        sim.step(1)
    a = lists(sims[0], md.MD_NL_CELL_WAVES, nl_block=nl_block)
    b = lists(sims[1], md.MD_NL_LANES)
    assert (b >= 0).sum() > 50 * len(pos)
    assert np.array_equal(a, b)
