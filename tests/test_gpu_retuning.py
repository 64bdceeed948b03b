"""A change of the force pass's lanes or workgroup alone leaves a list that stands as it
is: md_forces and md_step follow with no new list, also where the automatic tile
shape for the new lanes is another one; the next build takes that one.  Forces to
1e-12 of the largest (sums in another order), lists and, with the same tuning,
steps bit for bit."""
import numpy as np
import pytest

from gpu_helpers import state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

# systems whose automatic shape changes with the lanes
CASES = [(8500, 4, 64), (30000, 1, 64), (30000, 2, 192), (16000, 8, 128)]


def shape(sim):
    t = sim.get_tuning()
    return t["tile_cells"], t["tile_y"], t["tile_z"]


@pytest.mark.parametrize("reorder", [True, False])
@pytest.mark.parametrize("n,lanes,block", CASES)
def test_lanes_alone_keep_the_list(n, lanes, block, reorder):
    L, pos, vel = state(n, 0.8442, 107, jitter=0.05)
    sim = md.Simulation(pos, vel, L, r_cut=2.5, dt=0.004, reorder=reorder)
    sim.prepare()
    f, cnt, first = sim.state()["f"], sim.nl_counts(), shape(sim)
    sim.set_tuning(force_lanes=lanes, force_block=block)
    assert shape(sim) == first
    sim.forces()
    d = np.abs(sim.state()["f"] - f).max()
    assert d <= 1e-12 * np.abs(f).max()
    assert np.array_equal(sim.nl_counts(), cnt)
    other = md.Simulation(pos, vel, L, r_cut=2.5, dt=0.004, reorder=reorder)
    other.set_tuning(force_lanes=lanes, force_block=block)
    assert shape(other) != first
    other.prepare()
    for x in (sim, other):
        x.step(15, 5)
    a, b = sim.state(), other.state()
    for k in ("pos", "vel", "f"):
        assert np.array_equal(a[k], b[k]), k
    sim.prepare()
    assert shape(sim) == first  # the forces were computed with it
    sim.set_tuning(force_lanes=lanes, force_block=block)
    sim.prepare()
    assert shape(sim) == shape(other)
    other.prepare()
    assert np.array_equal(sim.state()["f"], other.state()["f"])


def test_batches_take_the_new_shape_at_once():
    L, pos, vel = state(30000, 0.8442, 107, jitter=0.05)
    sy = dict(pos=pos, vel=vel, L=L, r_cut=2.5, dt=0.004, skin=0.3)
    a, b = (md.Batch([sy, sy], precision="fp64") for _ in range(2))
    a.prepare()
    for x in (a, b):
        x.set_tuning(force_lanes=8, force_block=64)
        x.prepare()
        x.run(12)
    assert a.get_tuning() == b.get_tuning()
    for r in range(2):
        assert np.array_equal(a.state(r)["pos"], b.state(r)["pos"])
