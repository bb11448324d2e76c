"""The estimate behind the server's turns, compiled from its header with the
host compiler: a simulation is charged for the contraction it really takes,
so that turns have about the same device time whatever the coupling."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_11169_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "step_cost.hpp"
int main() {
    icwf_config c{};
    c.n_traj = 500; c.n_r = 512; c.n_R = 256;
    for (int prec : {ICWF_PREC_FP64, ICWF_PREC_MIXED}) {
        c.precision = prec;
        std::printf("%.17g %.17g %.17g %.17g\n", icwf::step_cost_ms(c, ICWF_CONTRACTION_TABLE, 0),
                    icwf::step_cost_ms(c, ICWF_CONTRACTION_PRODUCTS, 28), icwf::step_cost_ms(c, ICWF_CONTRACTION_BILINEAR, 1),
                    icwf::step_cost_ms(c, ICWF_CONTRACTION_FP32, 48));
    }
    std::printf("%d %d %d %d\n", icwf::turn_steps(10, 4.0, 4.0, 100), icwf::turn_steps(10, 4.0, 1.0, 100),
                icwf::turn_steps(10, 4.0, 1.0, 25), icwf::turn_steps(10, 1e9, 1e-3, 2000000000));
}
"""


def test_cost_follows_the_route(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "cost.cpp", tmp_path / "cost"
    src.write_text(DRIVER)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    lines = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines()
    assert lines[0] == lines[1]                       # the route, not the form asked for
    table, products, bilinear, fp32 = (float(x) for x in lines[0].split())
    pairs = 512 * 513 / 2
    per_flop = 1 / 4e10
    assert table - bilinear == pytest.approx(4 * pairs * 512 * 256 * per_flop)
    assert products - bilinear == pytest.approx(4 * pairs * (512 + 256) * 32 * per_flop)
    assert fp32 - bilinear == pytest.approx(4 * pairs * (512 * 256 / 2 + (512 + 256) * 48) * per_flop)
    assert lines[2] == "10 40 25 1000000"


def test_the_server_asks_the_simulation():
    """The cost is set from the created simulation's route, never from the submitted configuration alone."""
    server = open(os.path.join(CSRC, "icwf_server.cpp")).read()
    assert server.count("step_cost_ms(") == 1 and "step_cost_ms(rq->cfg, route, rank)" in server
    assert "icwf_contraction_route(sim, &route)" in server and "icwf_contraction_rank(sim, &rank)" in server
