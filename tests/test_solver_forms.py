"""The FP64 gas-kinetic solvers against their moment form in long double
(host build of the library's own routines, tests/solver_forms.cpp): Euler and
Navier-Stokes, subsonic and supersonic, smooth and jumping data, no jump at
all (tau = 0), collision times from far below to far above the time step."""
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
    out = str(tmp_path_factory.mktemp("forms") / "forms")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-ffp-contract=on", "--cuda-host-only", "-x", "hip",
                    os.path.join(HERE, "solver_forms.cpp"), "-o", out], check=True, capture_output=True)
    return out


@pytest.mark.parametrize("dim", [1, 2])
def test_primitive_form_matches_moment_form(exe, dim):
    cases = list(itertools.product([0.0, 1e-3, 1.0], [0.2, 3.0], [0.0, 1e-3, 0.3], [1e-4, 1e-2]))
    text = "".join(f"{dim} {mu} {mach} {jump} {dt} 2000 {n}\n" for n, (mu, mach, jump, dt) in enumerate(cases))
    out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.split()
    assert len(out) == len(cases)
    for case, w in zip(cases, out):
        assert float(w) <= 1.0, (dim, case, w)
