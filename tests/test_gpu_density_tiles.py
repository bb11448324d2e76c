"""Densities and norm by every tile size of the wavefunction's product (16 and
32 grid points, ragged trajectory counts), at t = 0 against the sums
written out in NumPy from the state read back.

Bars: an entry of Psi = sum_a C_a psi1^a psi2^a is off by at most
d = 2 (N + 8) eps sum_a |C_a psi1^a psi2^a| on either side, so a density by at
most hR sum_j (2 |Psi| 2 d + (2 d)^2) plus n_R + 8 roundings of itself."""

import numpy as np
import pytest

from paper_1805_11169_amd import icwf, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,n_r,n_R", [(1, 32, 32), (37, 64, 32), (64, 512, 256), (65, 256, 1024), (130, 1024, 256),
                                       (70, 4096, 512), (20, 4096, 32)])
def test_tiles(N, n_r, n_R):
    print(f"[case] densities N={N} on {n_r} x {n_R}", flush=True)
    wl = inputs.gaussian_basis(N, n_r=n_r, n_R=n_R, seed=N)
    sim = icwf.Simulation.from_workload(wl, C0=wl.extra["C0"])
    obs, st = sim.observables(), sim.state()
    sim.close()
    hr, hR = (wl.r_max - wl.r_min) / n_r, (wl.R_max - wl.R_min) / n_R
    U = st["C"][:, None] * st["psi1"]
    Psi = np.abs(U.T @ st["psi2"])
    eps = np.finfo(float).eps
    d = 4 * (N + 8) * eps * (np.abs(U).T @ np.abs(st["psi2"]))
    off = 2 * Psi * d + d * d
    for got, axis, h, n in ((obs["rho_r"], 1, hR, n_R), (obs["rho_R"], 0, hr, n_r)):
        ref = h * (Psi * Psi).sum(axis)
        assert np.all(np.abs(got - ref) <= h * off.sum(axis) + (n + 8) * eps * ref)
    ref = hr * hR * (Psi * Psi).sum()
    assert abs(obs["norm"] - ref) <= hr * hR * off.sum() + (n_r + n_R + 16) * eps * ref
