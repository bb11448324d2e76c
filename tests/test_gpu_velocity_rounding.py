"""Rounding of the Bohmian velocities (Eqs. 10-11), in both of their kernels.

One CWF carries the ansatz (C = e_0), so v = Im(psi' / psi) / m of that CWF:
the sums of its samples with the periodic sinc and derivative tables and
nothing else.  The terms of the derivative alternate in sign, so their order
decides the error.  Bar: the median error over the trajectories, against long
double, is at most 1.25 times that of the same sums taken point by point (in
FP64 with fused multiply-adds, emulated here; the median of 500 samples
scatters by a tenth).  Sums that take every second point first leave 1.4 to
2.0 times it."""

import numpy as np
import pytest

from paper_1805_11169_amd import icwf, inputs

pytestmark = pytest.mark.gpu

PI = np.longdouble("3.14159265358979323846264338327950288")


def _tables(xq, x_min, h, n):
    """Periodic sinc and its derivative at xq in long double, rounded to FP64 (the entry of the
    nearest point of the derivative from the others, as a constant has none)."""
    u = ((xq.astype(np.longdouble) - x_min) / h)[:, None] - np.arange(n)[None, :]
    t = PI * u / n
    s, c = np.sin(PI * u), np.cos(PI * u)
    S = s / (n * np.tan(t))
    D = (PI * c / (n * np.tan(t)) - s * (PI / n) / (n * np.sin(t) ** 2)) / h
    rows, near = np.arange(len(xq)), np.abs(np.remainder(u + n / 2, n) - n / 2).argmin(1)
    D[rows, near] = 0
    D[rows, near] = -D.sum(1)
    return S, D


def _chain(T, psi):
    """sum_i T[:, i] psi_i point by point with fused multiply-adds in FP64."""
    re, im = np.zeros(len(T)), np.zeros(len(T))
    for i in range(T.shape[1]):
        t = T[:, i].astype(np.longdouble)
        re = (re + t * psi[i].real).astype(np.float64)
        im = (im + t * psi[i].imag).astype(np.float64)
    return re + 1j * im


# per species: points, box, width, momentum and centre of the CWF
R_GRIDS = [((1024, (-50.0, 50.0), 3.0, 0.2, 0.4), (256, (-9.0, 9.0), 0.38, 0.3, -4.0)),
           ((512, (-75.0, 75.0), 6.0, 0.05, 1.0), (256, (-20.0, 20.0), 1.5, 0.2, -3.0))]


@pytest.mark.parametrize("N", [500, 640])       # small ensembles have a kernel of their own up to 576
@pytest.mark.parametrize("species", R_GRIDS)
def test_velocities_round_as_sums_in_order(N, species):
    g = np.random.default_rng(5)
    (n_r, r_box, *_), (n_R, R_box, *_) = species
    wl = inputs.gaussian_basis(N, n_r=n_r, n_R=n_R, r_box=r_box, R_box=R_box, model=inputs.MODEL_CAVITY, seed=1)
    at = []
    for (n, box, width, k, centre), psi in zip(species, (wl.psi1, wl.psi2)):
        h = (box[1] - box[0]) / n
        x = box[0] + h * np.arange(n)
        f = np.exp(-((x - centre) / width) ** 2 / 2 + 1j * k * x)
        psi[:] = f / np.sqrt(h * np.sum(abs(f) ** 2))
        at.append(centre + 0.7 * width * g.standard_normal(N))
    wl.r0[:], wl.R0[:] = at
    C = np.zeros(N, complex)
    C[0] = 1.0
    print(f"[case] velocities of one CWF at {N} positions, {n_r} x {n_R}", flush=True)
    sim = icwf.Simulation.from_workload(wl, C0=C)
    got = sim.velocities()[:2]
    sim.close()
    for v, xq, (n, box, *_), psi, m in zip(got, at, species, (wl.psi1[0], wl.psi2[0]), (wl.m_r, wl.m_R)):
        h = (np.longdouble(box[1]) - np.longdouble(box[0])) / n
        S, D = _tables(xq, np.longdouble(box[0]), h, n)
        p = psi.astype(np.clongdouble)
        exact = np.imag((D @ p) / (S @ p))
        chain = np.imag(_chain(D.astype(np.float64), psi) / _chain(S.astype(np.float64), psi))
        ours, theirs = (float(np.median(np.abs(e - exact))) for e in (v * m, chain))
        print(f"[result] {n} points: library {ours:.2e}, in order {theirs:.2e}", flush=True)
        assert ours < 1.25 * theirs
