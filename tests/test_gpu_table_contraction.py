"""The contractions that keep the W_c table: in FP64 and, less a short sum of
products, in FP32 (the mixed form).  Sharp Shin-Metiu couplings (small R_f),
for which no sum of products pays; every case asserts that it takes the route
it is about.

Bars: in FP64 1e-12 of the largest entry, as for the matrices everywhere; with
the FP32 pass 1e-5 of the sum of moduli of what it adds (a chain of 64
products of roundings of 6e-8), so that a pass that added nothing, or from
CWFs of another step, would be far outside."""

import numpy as np
import pytest

from oracle import icwf as oicwf
from paper_1805_11169_amd import icwf, inputs

from oracle_runs import init_for, rel_max, setup_for, wc_table

pytestmark = pytest.mark.gpu

L, R_L, R_R = 19.0, 3.1, 4.0
TABLE, FP32 = icwf.CONTRACTION_TABLE, icwf.CONTRACTION_FP32
FORM = {TABLE: icwf.PREC_FP64, FP32: icwf.PREC_MIXED}


def _workload(N, n_r, n_R, R_f, seed=17, **kw):
    return inputs.gaussian_basis(N, n_r=n_r, n_R=n_R, model=inputs.MODEL_SHIN_METIU, params=[L, R_f, R_L, R_R],
                                 seed=seed, **kw)


def _simulation(wl, route, **kw):
    sim = icwf.Simulation.from_workload(wl, precision=FORM[route], C0=wl.extra["C0"], **kw)
    assert sim.contraction_route() == route
    return sim


def _residual(table, terms):
    """What the first `terms` products of the cross approximation (largest
    remaining entry as pivot) leave of the table."""
    W = table.copy()
    for _ in range(terms):
        i, j = np.unravel_index(np.abs(W).argmax(), W.shape)
        W -= np.outer(W[:, j], W[i] / W[i, j])
    return W


def _check(wl, sim, route, pairs=None):
    """Entries of Wc and K at (b, a), b <= a, against those of the simulation's
    own CWFs and positions; returns its state."""
    s = setup_for(wl)
    S, K, Wc = sim.matrices()
    state = sim.state()
    N = wl.n_traj
    if pairs is None:
        g = np.random.default_rng(N)
        pairs = [tuple(sorted(p)) for p in g.integers(0, N, (40, 2))] + [(N - 1, N - 1), (0, N - 1), (N - 2, N - 1)]
        pairs += [(a, a) for a in g.integers(0, N, 20)]
        overlaps = np.argsort(-np.abs(np.triu(S, 1)).ravel())       # and the pairs that overlap most
        pairs += [divmod(int(e), N) for e in overlaps[np.r_[0:20, g.integers(20, 20 * N, 40)]]]
    table = wc_table(s)
    full = s.model.W(s.r[:, None], s.R[None, :])
    res = np.abs(_residual(table, sim.contraction_rank())) if route == FP32 else None
    err = err_k = added = 0.0
    for b, a in pairs:
        P1 = np.conj(state["psi1"][b]) * state["psi1"][a] * s.hr
        P2 = np.conj(state["psi2"][b]) * state["psi2"][a] * s.hR
        k = P1 @ full @ P2 - P1 @ s.model.W(s.r, state["R"][a]) * P2.sum() - P1.sum() * (s.model.W(state["r"][a], s.R) @ P2)
        err = max(err, abs(Wc[b, a] - P1 @ table @ P2))
        err_k = max(err_k, abs(K[b, a] - k))
        if route == FP32:
            added = max(added, np.abs(P1) @ res @ np.abs(P2))
    size = np.max(np.abs(Wc))
    bar = 1e-12 * size
    if route == FP32:
        bar = 1e-5 * added + 1e-14 * size
        assert added > 1e-8 * size                          # the pass has something to add
    print(f"[result] of max |Wc|: Wc {err / size:.2e} K {err_k / size:.2e} bar {bar / size:.2e} FP32 part {added / size:.2e}",
          flush=True)
    assert err < bar and err_k < 4 * bar + 1e-12 * np.max(np.abs(K))
    return state


# (n_r, n_R, N, R_f): one and several chunks and tiles of the FP32 pass (64 x 64), ragged N, more tiles than work-groups
GRIDS = [(64, 64, 37, 2.0), (128, 256, 130, 0.2), (512, 128, 70, 0.3), (256, 128, 530, 0.5)]


@pytest.mark.parametrize("route", [TABLE, FP32])
@pytest.mark.parametrize("n_r,n_R,N,R_f", GRIDS)
def test_contraction_at_the_start(n_r, n_R, N, R_f, route):
    print(f"[case] table on {n_r} x {n_R}, N={N} R_f={R_f} route={route}", flush=True)
    wl = _workload(N, n_r, n_R, R_f)
    sim = _simulation(wl, route)
    _check(wl, sim, route, None if N > 100 else [(b, a) for a in range(N) for b in range(a + 1)])
    sim.close()


@pytest.mark.parametrize("propagator", [icwf.PROP_SPLIT, icwf.PROP_CRANK_NICOLSON])
def test_fp32_pass_follows_the_cwfs(propagator):
    """Both propagators keep the FP32 copy of psi1 current: the contraction of
    the CWFs after each of a few steps, and observables within the mixed bar."""
    print(f"[case] FP32 pass over steps, propagator {propagator}", flush=True)
    wl = _workload(70, 256, 128, 0.5)
    sim = _simulation(wl, FP32, propagator=propagator)
    for _ in range(3):
        sim.step(2)
        state = _check(wl, sim, FP32)
    o = sim.observables()
    sim.close()
    assert np.max(np.abs(state["psi1"] - wl.psi1)) > 1e-3        # they have moved
    setup = setup_for(wl)
    if propagator == icwf.PROP_CRANK_NICOLSON:
        setup.propagator = "cn"
    _, hist = oicwf.run(setup, init_for(setup, wl), 6)
    ref = hist[-1]
    assert abs(o["norm"] - ref["norm"]) < 1e-5 * abs(ref["norm"])
    for key in ("rho_r", "rho_R", "r", "R"):
        assert rel_max(o[key], ref[key]) < 1e-5, key


@pytest.mark.parametrize("route", [TABLE, FP32])
def test_batch_is_each_alone(route):
    import torch
    print(f"[case] batch of three that keep the table, route {route}", flush=True)
    wls = [_workload(100, 256, 128, R_f, seed=s) for s, R_f in ((1, 0.5), (2, 0.52), (3, 0.55))]
    alone = []
    for wl in wls:
        sim = _simulation(wl, route)
        sim.step(3)
        alone.append(sim.state())
        sim.close()
    stream = torch.cuda.Stream()
    sims = [_simulation(wl, route, stream=stream) for wl in wls]
    icwf.step_batch(sims, 3)
    for sim, a in zip(sims, alone):
        b = sim.state()
        assert all(np.array_equal(a[k], b[k]) for k in ("r", "R", "psi1", "psi2", "C"))
        sim.close()


# (N, n_r, n_R, solver): the integrals beside the contraction for the room there is (n_r n_R >= 256 N) or, in FP64,
# for want of explicit inverses (asked for, or N no power of two); or ahead of the fork
FORKED = [(1024, 512, 512, icwf.SOLVER_AUTO), (1024, 256, 128, icwf.SOLVER_TRIANGULAR),
          (1100, 256, 128, icwf.SOLVER_AUTO), (1024, 256, 128, icwf.SOLVER_AUTO)]


@pytest.mark.parametrize("route", [TABLE, FP32])
@pytest.mark.parametrize("N,n_r,n_R,solver", FORKED)
def test_forked_step(N, n_r, n_R, solver, route):
    """Steps that fork with a table contraction, replayed and launched kernel
    by kernel: bitwise alike, and the matrices those of the CWFs and positions
    they end with (split tiles at the end of the queues among them)."""
    print(f"[case] forked step N={N} {n_r} x {n_R} solver={solver} route={route}", flush=True)
    wl = _workload(N, n_r, n_R, 0.8 if n_R == 512 else 0.5)
    ends = []
    for timing in (False, True):
        sim = _simulation(wl, route, solver=solver)
        if timing:
            sim.set_timing(True)
        sim.step(3)
        sim.sync()
        ends.append(_check(wl, sim, route) if not timing else sim.state())
        sim.close()
    assert all(np.array_equal(ends[0][k], ends[1][k]) for k in ("r", "R", "psi1", "psi2", "C"))
