"""Results copied out of device memory are ordinary arrays of their own, also
where the copy goes through page-locked memory: there in a forked child,
holding no pages down, zeros until they are written."""

import os

import numpy as np
import pytest

from paper_1805_11169_amd import icwf, inputs

pytestmark = pytest.mark.gpu


def _flags(a):
    """VmFlags of the mapping that holds the middle of the array."""
    addr = a.ctypes.data + a.nbytes // 2
    inside = False
    for line in open("/proc/self/smaps"):
        word = line.split()
        if word[0] == "VmFlags:":
            if inside:
                return word[1:]
        elif "-" in word[0]:
            lo, hi = (int(x, 16) for x in word[0].split("-"))
            inside = lo <= addr < hi
    raise AssertionError("no mapping")


def _is_ordinary(a):
    assert a.flags.owndata or a.base.flags.owndata
    assert not {"dc", "io", "pf"} & set(_flags(a))      # left out of a fork; device memory


def _propagator(n_r, n_R):
    wl = inputs.shin_metiu(4, n_r=n_r, n_R=n_R, n_bo=0)
    psi0 = np.random.default_rng(n_r).standard_normal((n_r, n_R)) + 1j
    return icwf.ExactPropagator(icwf.config_from_workload(wl), psi0), psi0


# 8, 16, 32 and 64 MiB: plain, at the two ends of the staged sizes, plain
@pytest.mark.parametrize("n_r,n_R", [(1024, 512), (1024, 1024), (4096, 512), (4096, 1024)])
def test_wavefunctions(n_r, n_R):
    print(f"[case] wavefunctions of {n_r} x {n_R} points", flush=True)
    x, psi0 = _propagator(n_r, n_R)
    got = [x.psi() for _ in range(3)]                   # kept together: none is another's memory
    x.close()
    for p in got:
        assert np.array_equal(p, psi0)
        _is_ordinary(p)
    got[0][:] = 0
    assert np.array_equal(got[1], psi0) and np.array_equal(got[2], psi0)


def test_a_forked_child_reads_a_result():
    x, psi0 = _propagator(2048, 512)
    p = x.psi()
    x.close()
    _is_ordinary(p)
    child = os.fork()
    if child == 0:
        os._exit(0 if np.array_equal(p, psi0) else 1)
    assert os.waitpid(child, 0)[1] == 0


def test_state_and_matrices():
    wl = inputs.gaussian_basis(1024, n_r=512, n_R=64, seed=2)
    print("[case] state and matrices of N = 1024", flush=True)
    sim = icwf.Simulation.from_workload(wl, C0=wl.extra["C0"])
    state, matrices = sim.state(), sim.matrices()
    sim.close()
    assert np.array_equal(state["psi1"], wl.psi1) and np.array_equal(state["psi2"], wl.psi2)
    assert all(np.abs(m - m.conj().T).max() < 1e-12 * np.abs(m).max() for m in (matrices[0], matrices[2]))
    for a in (state["psi1"], state["psi2"], *matrices):
        _is_ordinary(a)


def test_basis_of_a_refused_call_is_zeros():
    cfg = icwf.config_from_workload(inputs.shin_metiu(4, n_r=4096, n_R=32, n_bo=0))
    R = np.linspace(-8.0, 8.0, 256)                     # 16 MiB of states
    print("[case] BO basis, 4096 points, 256 values", flush=True)
    states, _, info = icwf.bo_states(cfg, R, 2, max_iter=3, tol=1e-300, check=False)
    assert info["status"] == icwf.ESOLVE and np.all(np.abs(states).max(axis=2) > 0)
    _is_ordinary(states)
    R[5] = np.nan
    states, energies, info = icwf.bo_states(cfg, R, 2, check=False)
    assert info["status"] == icwf.ENONFINITE and not states.any() and not energies.any()


def test_kept_results_hold_no_page_locked_memory():
    import torch
    stats = getattr(torch.cuda, "host_memory_stats", None)
    if stats is None:
        pytest.skip("this PyTorch does not count page-locked memory")
    x, _ = _propagator(2048, 512)
    kept = [x.psi()]
    locked = stats()["allocated_bytes.current"]         # (its count of active bytes never falls)
    kept += [x.psi() for _ in range(6)]
    x.close()
    assert stats()["allocated_bytes.current"] == locked
