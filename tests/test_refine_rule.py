"""When a mixed-precision refinement ends (csrc/refine_rule.h), on the CPU.

The rule is compiled from the library's own header.  A simulated refinement
contracts the error by a factor c per sweep; the status word's bound is formed
from the residual BEFORE a sweep's correction, so it is about the size of that
correction.  Whatever c is, a column that ends without having stalled must
have a bound the status word accepts.
"""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_0912_2572_amd", "csrc")

SOURCE = """
#include "refine_rule.h"
extern "C" int state(double rel, double prev, int sweeps, double tol) {
    return tsqr::refine_state(rel, prev, sweeps, tol);
}
extern "C" int done(int st, double tol, int known, double eta) {
    return tsqr::refine_done(tsqr::RefineState(st), tol, known != 0, eta);
}
extern "C" double eta_max() { return tsqr::kEtaMax; }
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    src, lib = d / "rule.cpp", d / "rule.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)], check=True)
    L = ctypes.CDLL(str(lib))
    L.state.argtypes = [ctypes.c_double, ctypes.c_double, ctypes.c_int, ctypes.c_double]
    L.done.argtypes = [ctypes.c_int, ctypes.c_double, ctypes.c_int, ctypes.c_double]
    L.eta_max.restype = ctypes.c_double
    return L


def refine(L, c, tol, first=True, max_sweeps=30):
    """Corrections 1, c, c^2, ... down to rounding; returns (sweeps, bound, stalled)."""
    prev, err = 1.0, 1.0
    for s in range(max_sweeps):
        eta = max(err, 1e-17)              # the residual pass of this sweep
        rel = max(err, 1e-16)              # its correction
        st = L.state(rel, prev, s, tol)
        if L.done(st, tol, int(first or s > 0), eta):
            return s + 1, eta, st == 2
        prev, err = rel, err * c
    return max_sweeps, eta, True


def test_a_column_that_did_not_stall_is_never_flagged(rule):
    for c in np.logspace(-16, -0.2, 400):
        sweeps, bound, stalled = refine(rule, float(c), 1e-14)
        assert stalled or bound <= rule.eta_max(), c
        # no more than one sweep past the first whose estimate is below tol
        first = next(s for s in range(1, 400) if c * c ** s <= 1e-14 or c ** s < 1e-16)
        assert sweeps <= first + 2, c


def test_both_sides_of_the_single_correction_threshold_agree(rule):
    lo, hi = refine(rule, 0.99e-7, 1e-14), refine(rule, 1.01e-7, 1e-14)
    assert lo[0] == hi[0] == 3 and max(lo[1], hi[1]) <= rule.eta_max()


def test_a_loose_tolerance_alone_decides(rule):
    assert refine(rule, 1e-4, 1e-6)[0] == 2
    assert refine(rule, 1e-4, 1e-6, first=False)[0] == 2


def test_stall_and_nan_end_a_column(rule):
    assert rule.state(0.5, 0.52, 1, 1e-14) == 2
    assert rule.state(float("nan"), 1.0, 0, 1e-14) == 2
    assert rule.done(2, 1e-14, 0, float("nan")) == 1


def test_zero_solution_waits_for_its_residual_pass(rule):
    st = rule.state(0.0, 1.0, 0, 1e-14)
    assert st == 1 and rule.done(st, 1e-14, 0, 0.0) == 0 and rule.done(st, 1e-14, 1, 0.0) == 1
