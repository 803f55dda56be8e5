"""Host test of the FP64 reciprocal, reciprocal square root and square root
that the pair terms use: their errors in units in the last place, from
approximations off by up to 2^-24 (the hardware's are better).  Derived bounds:
a correction whose own terms are below 2^-70 leaves the final operation's rounding
(half a unit) for the reciprocal and, with its exact residual, the square root,
and that of the product x y besides for the reciprocal square root (one unit
together).  The margin is the reference's own rounding (80-bit)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if not (shutil.which(HIPCC) or os.path.exists(HIPCC)):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("math") / "libmath_error.so")
    subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-host-only", "-fPIC", "-shared", "-mfma",
                    "-ffp-contract=on", "-I" + os.path.join(ROOT, "paper_1909_04504_amd", "csrc"),
                    "-o", out, os.path.join(ROOT, "tests", "native", "math_error.hip")], check=True)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("lo,hi", [(-60, 20), (-1, 1), (-1000, -900), (900, 1000)])
def test_errors_in_last_place(lib, lo, hi):
    worst = (ctypes.c_double * 3)()
    lib.math_error(ctypes.c_int64(400000), ctypes.c_uint64(7), lo, hi, 24, worst)
    rcp, rsqrt, sqrt = np.array(worst)
    assert rcp <= 0.51 and sqrt <= 0.51 and rsqrt <= 1.01
