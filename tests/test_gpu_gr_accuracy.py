"""The soft g(r)'s gradient against the same sums in 80-bit arithmetic, where a
pair reaches hundreds of narrow bins: an exponential formed from the one of the
bin before would be off by the square of the bins a pair reaches times the
rounding (1e-12 here).

One bin alone has a weight, and dt is so small that the steps add nothing
(dt^2 J / m < 1e-15), so the gradient is the bin's own.  Tolerance: a partner
staged as a shifted image is rounded by half an ulp of 2 L per coordinate,
3.1e-15 in r; t exp(-t^2 / 2 w^2) changes by at most 1.6 (dr / w) of its peak."""
import numpy as np
import pytest
import torch

from gpu_helpers import state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu


def reference(pos, L, bins, rmax, w, b):
    ld = np.longdouble
    pos, w = pos.astype(ld), ld(w)
    n = len(pos)
    rb = (ld(b) + ld(0.5)) * ld(rmax) / ld(bins)
    norm = ld(n) * ld(n) / ld(L) ** 3 * 4 * ld(np.pi) * rb * rb
    g = np.zeros((n, 3), ld)
    for i in range(n):
        d = pos[i] - pos
        d -= ld(L) * np.rint(d / ld(L))
        r = np.sqrt((d * d).sum(1))
        t = r - rb
        m = (np.abs(t) < 3 * w) & (np.arange(n) != i)
        f = -t[m] / (w * w) * np.exp(-0.5 * (t[m] / w) ** 2) / (w * np.sqrt(2 * ld(np.pi)))
        g[i] = (2 * f / norm / r[m]) @ d[m]
    return g


@pytest.mark.parametrize("bins,rmax,width,b", [(1024, 2.0, 0.2, 700), (1024, 1.59, 0.4, 900),
                                               (50, 2.5, 0.05, 22)])
def test_gradient_of_one_bin(bins, rmax, width, b):
    L, pos, vel = state(2200, 0.8, 83, jitter=0.05)
    sim = md.Simulation(pos, vel, L, r_cut=2.5, dt=1e-9, skin=0.3, reorder=False)
    sim.traj_forward(1, 1, bins, rmax, width)
    gobs = torch.zeros(1 + bins, dtype=torch.float64)
    gobs[1 + b] = 1.0
    gx, _, _ = sim.traj_backward(gobs)
    ref = reference(sim.state()["pos"], L, bins, rmax, width, b)
    err = np.linalg.norm(gx.cpu().numpy() - ref.astype(float)) / float(np.linalg.norm(ref.astype(float)))
    print(f"bins {bins} width {width}: {err:.2e}")
    assert err <= 1.6 * 3.1e-15 / width
