"""The distance bounds behind the sole-component rule of the Langevin kernels, compiled for the host from the kernels' own header: over any
number of steps the slack stays at or below what is left of it and the distance at or above what was walked, also where a
step is below the last bit of either."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "sole_bound.h"
extern "C" void walk(float* slack, float* rho, float by, long steps, int window) {
  SoleBound s;
  s.slack = *slack;
  s.rho = *rho;
  for (long i = 1; i <= steps; ++i) {
    s.moved(by);
    if (i % window == 0) s.window_ended(0.f);
  }
  *slack = s.slack;
  *rho = s.rho;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    d = tmp_path_factory.mktemp("sole")
    (d / "w.cpp").write_text(SOURCE)
    lib = str(d / "w.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2501_05370_amd", "csrc"),
                    str(d / "w.cpp"), "-o", lib], check=True)
    fn = ctypes.CDLL(lib).walk
    fn.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.POINTER(ctypes.c_float), ctypes.c_float, ctypes.c_long, ctypes.c_int]

    def run(slack, by, steps, window):
        s, r = ctypes.c_float(slack), ctypes.c_float(slack)
        fn(s, r, by, steps, window)
        return s.value, r.value
    return run


@pytest.mark.parametrize("window", [1, 7, 64])
@pytest.mark.parametrize("share", [1e-2, 3e-5, 2.9e-7, 8.9e-8, 4e-8, 2e-8, 1e-9])
@pytest.mark.parametrize("slack", [1.0, 1.9999999, 3e-4, 7.3e9])
def test_roundings_do_not_add_up(walk, share, slack, window):
    """Above the truth by a tenth of the margin the slack is set with, whatever the number of steps."""
    slack = float(np.float32(slack))
    by = float(np.float32(slack * share))
    steps = min(1_000_000, int(0.95 / share)) // window * window
    got, rho = walk(slack, by, steps, window)
    assert got <= slack - steps * by + 1e-5 * slack
    assert rho >= slack + steps * by
    # and the bound is of use: 3e-5 of the distance a window at most
    lost = 3e-5 * (steps // window + 1)
    assert got >= (slack - steps * by) * (1 - lost) - lost * slack


def test_a_mixture_of_one_component_never_runs_out(walk):
    assert walk(float("inf"), 1.0, 1000, 8)[0] == float("inf")
