"""The reverse gas-kinetic solvers (host build of the library's own routines,
tests/adjoint_forms.cpp) against central differences of the forward moment
form in long double: Euler and Navier-Stokes, subsonic and supersonic, both
output sets (with and without values), collision times from far below to far
above the time step.

Bound 1e-7 of the largest adjoint of a solve: four-point differences of step
h = 5e-5 in long double are off by h^4 / 30 times fifth derivatives (2e-19
times up to 1e10 of the first, through exp(-dt / tau) at pressure jumps of a
few 1e-3) plus the forward's rounding over h, (tau / dt)^2 1e-19 / h in the
time coefficients: 2e-9 each at most times the sizes summed; the reverse's own
rounding enters as 64 eps of those sizes, which exceed the largest adjoint by
up to (1 + Mach)^4 / dt in its time derivative terms."""
import itertools
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("adjforms") / "adjforms")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-ffp-contract=on", "--cuda-host-only", "-x", "hip",
                    os.path.join(HERE, "adjoint_forms.cpp"), "-o", out], check=True, capture_output=True)
    return out


def test_reverse_solvers_match_differences(exe):
    cases = list(itertools.product([0.0, 1e-3, 1.0], [0.2, 3.0], [5e-3, 0.3], [1e-3, 1e-2]))
    text = "".join(f"{mu} {mach} {jump} {dt} 200 {n}\n" for n, (mu, mach, jump, dt) in enumerate(cases))
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.split("\n")
    for case, line in zip(cases, out[:len(cases)]):
        a, b = (float(v) for v in line.split())
        assert a <= 1e-7 and b <= 1e-7, (case, a, b)
