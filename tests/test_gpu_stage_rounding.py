"""Rounding of the RK4 stages (Eq. 8 amplifies it by up to 1 / (2 sqrt(eps))).

K v, whose sum has to stay a shallow one: real CWFs and real C make the first step's trajectories stand still, so
K(psi_1, x_0) is K(psi_1, x_1) and the whole RK4 step follows from the
library's own S and K before and after it; nearly orthogonal CWFs make S well
conditioned, so that nothing amplifies.  The step is repeated from these
matrices in long double, and in FP64 with K v summed by 256 lanes and a tree
and LAPACK's solves.  Bar: 1.5 times that one's error (N = 500 to 1984: one
chain of N / 4 terms in each of four lanes leaves 1.6 to 2.3 times)."""

import numpy as np
import pytest
import scipy.linalg

from paper_1805_11169_amd import icwf, inputs

pytestmark = pytest.mark.gpu


def _sum(P, n):
    """Row sums of P: a chain of every n-th column in each of n lanes, then a tree over them."""
    s = np.zeros((P.shape[0], n), complex)
    for k in range(0, P.shape[1], n):
        w = min(n, P.shape[1] - k)
        s[:, :w] += P[:, k:k + w]
    while s.shape[1] > 1:
        h = s.shape[1] // 2
        s = s[:, :h] + s[:, h:]
    return s[:, 0]


def _step(S, K, C, dt, lanes):
    """One RK4 step of Eq. 8 with K v summed by `lanes` lanes; 0: in long double."""
    def solver(A):
        cf = scipy.linalg.cho_factor(A, lower=True)
        if lanes:
            return lambda b: scipy.linalg.cho_solve(cf, b)
        Al = A.astype(np.clongdouble)

        def refined(b):
            x = scipy.linalg.cho_solve(cf, b.astype(complex)).astype(np.clongdouble)
            for _ in range(3):
                x = x + scipy.linalg.cho_solve(cf, (b - Al @ x).astype(complex))
            return x
        return refined

    def times(M, v):
        return _sum(M * v[None, :], lanes) if lanes else M.astype(np.clongdouble) @ v

    mid = 0.5 * (K[0] + K[1])
    A = [solver(S[0]), solver(0.5 * (S[0] + S[1])), solver(S[1])]
    k1 = -1j * A[0](times(K[0], C))
    k2 = -1j * A[1](times(mid, C + 0.5 * dt * k1))
    k3 = -1j * A[1](times(mid, C + 0.5 * dt * k2))
    k4 = -1j * A[2](times(K[1], C + dt * k3))
    return C + (dt / 6) * (k1 + 2 * k2 + 2 * k3 + k4)


def step_errors(N):
    """Relative errors of one step: the library's, and with 256-lane sums."""
    dt, eps = 1.0, 1e-8
    wl = inputs.gaussian_basis(N, n_r=256, n_R=128, r_box=(-40.0, 40.0), model=inputs.MODEL_SHIN_METIU, seed=N, dt=dt)
    g = np.random.default_rng(N)
    for psi, box, n in ((wl.psi1, (wl.r_min, wl.r_max), 256), (wl.psi2, (wl.R_min, wl.R_max), 128)):
        x = g.standard_normal(psi.shape)
        psi[:] = x / np.sqrt((x * x).sum(1, keepdims=True) * (box[1] - box[0]) / n)
    C = g.standard_normal(N).astype(complex)
    sim = icwf.Simulation.from_workload(wl, C0=C)
    assert wl.eps == eps
    S0, K0, _ = sim.matrices()
    before = sim.observables()
    sim.step(1)
    S1, K1, _ = sim.matrices()
    after = sim.observables()
    sim.close()
    assert np.array_equal(before["r"], after["r"]) and np.array_equal(before["R"], after["R"])
    reg = eps * np.eye(N)
    S, K = [S0 + reg, S1 + reg], [K0, K1]
    ref = _step(S, K, C.astype(np.clongdouble), dt, 0)

    def err(x):
        return float(np.sqrt(np.sum(np.abs(x - ref) ** 2) / np.sum(np.abs(ref) ** 2)))
    return err(after["C"]), err(_step(S, K, C, dt, 256))


@pytest.mark.parametrize("N", [500, 900, 1500, 1984])
def test_rounding_of_k_v(N):
    print(f"[case] one step of {N} nearly orthogonal CWFs, 256 x 128", flush=True)
    got, tree = step_errors(N)
    print(f"[result] N={N}: library {got:.2e}, 256 lanes and a tree {tree:.2e}", flush=True)
    assert got < 1.5 * tree


@pytest.mark.parametrize("N,n_r,n_R", [(250, 64, 32), (500, 128, 64)])
def test_rounding_of_the_solves(N, n_r, n_R):
    """C_0 = (S + eps I)^-1 b of nearly orthogonal CWFs (condition 3 to 4)
    against long double, mean of 8 ensembles: below 1.6 times LAPACK's error.
    An elimination that rounds an entry once for each column leaves 1.40 to
    1.45 times it, one that rounds it twice 1.74 to 1.76."""
    print(f"[case] solves of {N} nearly orthogonal CWFs, {n_r} x {n_R}", flush=True)
    errors = []
    for seed in range(8):
        wl = inputs.gaussian_basis(N, n_r=n_r, n_R=n_R, r_box=(-40.0, 40.0), model=inputs.MODEL_SHIN_METIU, seed=N)
        g = np.random.default_rng(100 * N + seed)

        def complex_normal(*shape):
            return g.standard_normal(shape) + 1j * g.standard_normal(shape)
        for psi, box, n in ((wl.psi1, (wl.r_min, wl.r_max), n_r), (wl.psi2, (wl.R_min, wl.R_max), n_R)):
            x = complex_normal(*psi.shape)
            psi[:] = x / np.sqrt((abs(x) ** 2).sum(1, keepdims=True) * (box[1] - box[0]) / n)
        wl.b0 = b = complex_normal(N)
        sim = icwf.Simulation.from_workload(wl)
        A = sim.matrices()[0] + wl.eps * np.eye(N)
        C = sim.observables()["C"]
        sim.close()
        cf, Al = scipy.linalg.cho_factor(A, lower=True), A.astype(np.clongdouble)
        lapack = scipy.linalg.cho_solve(cf, b)
        x = lapack.astype(np.clongdouble)
        for _ in range(3):
            x = x + scipy.linalg.cho_solve(cf, (b - Al @ x).astype(complex))
        errors.append([float(np.sqrt(np.sum(np.abs(c - x) ** 2) / np.sum(np.abs(x) ** 2))) for c in (C, lapack)])
    got, lapack = np.mean(errors, axis=0)
    print(f"[result] N={N}: library {got:.2e}, LAPACK {lapack:.2e}", flush=True)
    assert got < 1.6 * lapack
