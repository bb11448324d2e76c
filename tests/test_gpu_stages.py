"""The RK4 stages at the edges of their kernels (one block of 64 rows in one
work-group, several blocks handing their parts on): the coefficients after
two steps against the oracle, in the S norm (1e-10, as in the one-step parity
tests), alone and in a batch, where a simulation that stops on a node leaves
its blocks' neighbours none to wait for."""

import numpy as np
import pytest

from oracle import icwf as oicwf
from oracle import models
from paper_1805_11169_amd import icwf, inputs

pytestmark = pytest.mark.gpu


def _oracle(wl, steps):
    m = models.make("shin_metiu", wl.model_params)
    s = oicwf.Setup(m, wl.r_min, wl.r_max, wl.n_r, wl.R_min, wl.R_max, wl.n_R, wl.m_r, wl.m_R, wl.dt, wl.eps)
    st = oicwf.init(s, wl.r0, wl.R0, wl.psi1, wl.psi2, C0=wl.extra["C0"])
    for _ in range(steps):
        st = oicwf.step(s, st)
    return st


@pytest.mark.parametrize("N", [1, 63, 64, 65, 128, 129, 320])
def test_two_steps(N):
    wl = inputs.gaussian_basis(N, n_r=128, n_R=64, seed=N)
    print(f"[case] stages N={N}", flush=True)
    sim = icwf.Simulation.from_workload(wl, C0=wl.extra["C0"])
    sim.step(2)
    sim.sync()
    got = sim.state()["C"]
    sim.close()
    ref = _oracle(wl, 2)
    d = got - ref.C
    scale = np.sqrt(abs(np.conj(ref.C) @ ref.S @ ref.C))
    assert np.sqrt(abs(np.conj(d) @ ref.S @ d)) < 1e-10 * scale


@pytest.mark.parametrize("N", [64, 130])
def test_a_stopped_member_of_a_batch(N):
    import torch
    wls = [inputs.gaussian_basis(N, n_r=128, n_R=64, seed=s) for s in (1, 2, 3)]
    wls[1].psi2[:] = 0.0
    print(f"[case] batch of three, N={N}, one at a node", flush=True)
    alone = []
    for wl in (wls[0], wls[2]):
        sim = icwf.Simulation.from_workload(wl, C0=wl.extra["C0"])
        sim.step(3)
        alone.append(sim.state()["C"])
        sim.close()
    stream = torch.cuda.Stream()
    sims = [icwf.Simulation.from_workload(wl, stream=stream, C0=wl.extra["C0"]) for wl in wls]
    icwf.step_batch(sims, 3)
    with pytest.raises(icwf.ICWFError) as e:
        sims[1].sync()
    assert e.value.status == icwf.ENODE
    assert np.array_equal(sims[0].state()["C"], alone[0]) and np.array_equal(sims[2].state()["C"], alone[1])
    for s in sims:
        s.close()
