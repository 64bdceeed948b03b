"""The soft g(r) and its gradient at bins much narrower and much wider than the
kernel (successive bins by factors, or an exponential each), with more bins
than one word of lanes and a single one, against the oracle: g to 1e-9, as its
fixed-point sums are compared elsewhere, the gradient to 1e-8."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins,rmax,width", [(50, 2.5, 0.05), (300, 2.5, 0.05), (1024, 2.0, 0.2),
                                             (10, 2.0, 0.05), (9, 2.0, 0.05), (4, 2.0, 0.02),
                                             (1, 2.2, 0.1)])
@pytest.mark.parametrize("n", [1000, 4001])
def test_g_and_its_gradient(n, bins, rmax, width):
    L, pos, vel = state(n, 0.8, 71, jitter=0.05)
    sim = md.Simulation(pos, vel, L, r_cut=2.5, dt=0.004, skin=0.3, reorder=False)
    obs = sim.traj_forward(2, 1, bins, rmax, width).cpu().numpy()
    rng = np.random.default_rng(5)
    gobs = np.concatenate([[0.0], rng.standard_normal(bins)])
    gx, _, _ = sim.traj_backward(torch.tensor(gobs))
    s = oracle.make_sys(n, L, r_cut=2.5, skin=0.3, dt=0.004)
    ref = oracle.traj_adjoint(s, oracle.gr_spec(bins, rmax, width), 2, pos, vel, gobs[0], gobs[1:])
    assert np.abs(obs[1:] - ref["g"]).max() <= 1e-9 * max(1.0, np.abs(ref["g"]).max())
    d = np.linalg.norm(gx.cpu().numpy() - ref["grad_x0"])
    assert d <= 1e-8 * np.linalg.norm(ref["grad_x0"])
