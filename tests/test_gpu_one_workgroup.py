"""The cell build on both sides of the lines between one workgroup and the chain of
kernels (forced builds 5120 atoms; cells-only steps 12 288, dense ones 8192, with
reorder 4096): cells against the oracle, bit for bit, and steps against the
oracle's (positions to 1e-10, velocities to 1e-9, as the other short runs)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import WCA, check_cells, min_image, pair, state

pytestmark = pytest.mark.gpu

LJ, SOFT = (0.8442, 2.5), (0.8, WCA)


@pytest.mark.parametrize("n", [5120, 5121])
@pytest.mark.parametrize("nl", [True, False])
@pytest.mark.parametrize("rho,r_cut", [LJ, SOFT])
def test_forced_builds(n, nl, rho, r_cut):
    L, pos, vel = state(n, rho, 97, jitter=0.05)
    sim, s = pair(pos, vel, L, r_cut=r_cut, nl=nl, reorder=False)
    for _ in range(3):
        sim.build_cells()
        check_cells(sim, s, pos)


@pytest.mark.parametrize("n,rho,r_cut,reorder", [
    (8192, *LJ, False), (8193, *LJ, False), (12288, *SOFT, False), (12289, *SOFT, False),
    (4096, *SOFT, True), (4097, *SOFT, True), (4097, *LJ, True), (6000, 0.05, WCA, False),
])
def test_cells_only_steps(n, rho, r_cut, reorder):
    L, pos, vel = state(n, rho, 101, jitter=0.05)
    sim, s = pair(pos, vel, L, r_cut=r_cut, nl=False, reorder=reorder, dt=0.004)
    sim.prepare()
    sim.step(5, record_every=1)
    sim.step(6, record_every=1)
    p_ref, v_ref, _, o_ref, _ = oracle.run(s, pos, vel, 11)
    st, h = sim.state(), sim.history()
    assert np.abs(min_image(st["pos"] - p_ref, L)).max() < 1e-10
    assert np.abs(st["vel"] - v_ref).max() < 1e-9
    assert np.abs(h["U"] - o_ref["U"]).max() <= 1e-10 * np.abs(o_ref["U"]).max()
