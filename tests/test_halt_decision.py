"""A halt may be raised by another launch while a kernel runs (the
factorisations beside the contraction), so a work-group whose waves share a
unit of work or a ticket through LDS has to decide on it once: waves that each
read the flag for themselves part company, and those left behind then wait for
a unit nobody takes, or take one that was never written.

By reading the sources on the CPU; on the GPU a halt set from the host at
different moments of a forked step, where every kernel ends and the step
reports it."""

import os
import re
import time

import pytest

from paper_1805_11169_amd import icwf, inputs

CSRC = os.path.join(os.path.dirname(icwf.LIB_PATH), "csrc")


def _kernels():
    """(name, body) of every kernel under csrc/."""
    for f in sorted(os.listdir(CSRC)):
        if not f.endswith(".hip"):
            continue
        src = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, f)).read())
        for m in re.finditer(r"__global__", src):
            start = src.index("{", m.end())
            depth, end = 0, start
            for end in range(start, len(src)):
                depth += {"{": 1, "}": -1}.get(src[end], 0)
                if depth == 0:
                    break
            name = re.findall(r"(k_\w+)\s*\(", src[m.end():start])[0]
            yield f"{f}:{name}", src[start:end + 1]


def test_kernels_sharing_integers_decide_on_a_halt_once():
    sharing = {name: body for name, body in _kernels() if re.search(r"__shared__\s+int\b", body)}
    assert {"k_matrices.hip:k_wc", "k_matrices.hip:k_wc_sep", "k_solve.hip:k_rk_fwd",
            "k_solve.hip:k_rk_bwd"} <= set(sharing)
    for name, body in sharing.items():
        assert "flags[kFlagHalt]" not in body, name


@pytest.mark.gpu
@pytest.mark.parametrize("N,precision,R_f", [(1024, icwf.PREC_FP64, 5.0), (1024, icwf.PREC_FP64, 0.3),
                                             (1024, icwf.PREC_MIXED, 0.3), (1100, icwf.PREC_FP64, 5.0)])
def test_a_halt_during_a_forked_step_ends_it(N, precision, R_f):
    """256 x 128 grid (products, the dense table, the FP32 pass; stages through
    the explicit inverses and block by block): the flags of a failed
    factorisation written from another stream while steps are queued."""
    import torch
    wl = inputs.gaussian_basis(N, n_r=256, n_R=128, r_box=(-40.0, 40.0), model=inputs.MODEL_SHIN_METIU,
                               params=[19.0, R_f, 3.1, 4.0], seed=3)
    side = torch.cuda.Stream()
    for delay in (0.0, 0.5e-3, 1e-3, 2e-3, 4e-3):
        print(f"[case] halt {delay * 1e3} ms into 4 steps, N={N} R_f={R_f} precision={precision}", flush=True)
        sim = icwf.Simulation.from_workload(wl, precision=precision, C0=wl.extra["C0"])
        at = (-sim.ws.data_ptr()) % 256                      # the workspace begins with the status flags
        flags = sim.ws[at:at + 32].view(torch.int32)
        torch.cuda.synchronize()
        sim.step(4)
        t0 = time.perf_counter()
        while time.perf_counter() - t0 < delay:
            pass
        with torch.cuda.stream(side):
            flags[2].fill_(1)                                # a pivot that is not positive
            flags[0].fill_(1)                                # halt
        side.synchronize()
        with pytest.raises(icwf.ICWFError) as e:
            sim.sync()
        assert e.value.status == icwf.ESOLVE
        sim.close()
