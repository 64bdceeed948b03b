"""The cell-wave list build where the queues do not fit beside the staged atoms: alone,
in a batch, and in a batch where one replica has room for them and another has
not.  The lists' lengths and a run across rebuilds are those of the same systems
with their queues, bit for bit."""
import numpy as np
import pytest

from gpu_helpers import state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

# (atoms, density) of the replicas, and what they are tuned to: every stage at 155 KiB,
# or tiles of 64 cells, whose staged atoms fill the LDS in the dense replica alone
CASES = {
    "none_has_room": (((4000, 0.8442), (10976, 0.8442)), dict(stage_cap=6600)),
    "one_has_room": (((9300, 1.18), (6000, 0.4)), dict(tile_cells=4, tile_y=4, tile_z=4)),
}


@pytest.mark.parametrize("reorder", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_runs_without_queues(name, reorder):
    sizes, tuning = CASES[name]
    tuning = dict(tuning, nl_method=md.MD_NL_CELL_WAVES)
    systems = []
    for seed, (n, rho) in enumerate(sizes):
        L, pos, vel = state(n, rho, 5 + seed, jitter=0.05)
        systems.append(dict(pos=pos, vel=1.5 * vel, L=L, r_cut=2.5, dt=0.004, skin=0.3))
    b = md.Batch(systems, precision="fp64", reorder=reorder)
    b.set_tuning(**tuning)
    b.prepare()
    b.run(30)
    b.synchronize()
    for r, sy in enumerate(systems):
        alone = md.Simulation(sy["pos"], sy["vel"], sy["L"], r_cut=2.5, dt=0.004, skin=0.3,
                              reorder=reorder)
        full = md.Simulation(sy["pos"], sy["vel"], sy["L"], r_cut=2.5, dt=0.004, skin=0.3,
                             reorder=reorder)
        alone.set_tuning(**tuning)
        for sim in (alone, full):
            sim.prepare()
            sim.step(30)
        ref = full.state()
        assert full.reduce()["n_rebuilds"] > 0
        for got in (alone.state(), b.state(r)):
            for k in ("pos", "vel", "f"):
                assert np.array_equal(got[k], ref[k]), k
        assert np.array_equal(alone.nl_counts(), full.nl_counts())
        assert np.array_equal(b.nl_counts(r), full.nl_counts())
