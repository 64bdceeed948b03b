"""md_step with graphs on a stream that is being captured already cannot capture its
own: the call fails, launches nothing (what the outer capture holds changes nothing
when replayed) and leaves state and forces as they were, so the next call steps on
from there, bit for bit as if the failed one had not been made."""
import numpy as np
import pytest
import torch

from gpu_helpers import WCA, state
from paper_2003_14061_amd import md

pytestmark = pytest.mark.gpu

CASES = {
    "list": dict(n=4000, rho=0.8442, r_cut=2.5, dt=0.004),
    "cells": dict(n=4000, rho=0.8, r_cut=WCA, dt=0.005, neighbor_list=False),
    "half_list": dict(n=4000, rho=0.8442, r_cut=2.5, dt=0.004, newton3=True),
}


def same(a, b, rtol):
    for k in ("pos", "vel", "f"):
        assert np.allclose(a[k], b[k], rtol=rtol, atol=rtol * np.abs(b[k]).max()), k


@pytest.mark.parametrize("steps", [20, 21])
@pytest.mark.parametrize("name", list(CASES))
def test_a_refused_capture_leaves_the_state(name, steps):
    kw = dict(CASES[name])
    L, pos, vel = state(kw.pop("n"), kw.pop("rho"), 103, jitter=0.05)
    s = torch.cuda.Stream()
    sim = md.Simulation(pos, vel, L, stream=s, **kw)
    ref = md.Simulation(pos, vel, L, **kw)
    for x in (sim, ref):
        x.prepare()
    # (third-law forces add by atomics, to rounding)
    rtol = 1e-9 if kw.get("newton3") else 0.0
    before = sim.state()
    sim.set_graph(True)
    g = torch.cuda.CUDAGraph()
    mark = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s, capture_error_mode="relaxed"):
        mark += 1.0
        with pytest.raises(md.MDError) as e:
            sim.step(steps)
        assert e.value.status == -5
    g.replay()
    torch.cuda.synchronize()
    assert mark.eq(1.0).all()
    same(sim.state(), before, 0.0)
    for x in (sim, ref):
        x.step(steps, 1)
        x.step(steps, 1)
    same(sim.state(), ref.state(), rtol)
    assert len(sim.history()) == 2 * steps
