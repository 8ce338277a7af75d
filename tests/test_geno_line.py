"""The line reconstructions that settle smooth components from one ratio give
the bits of the general per-component routine (host build of the library's
own code, tests/geno_line.cpp)."""
import json
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def test_line_routines_match_per_component_routine(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "line")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-ffp-contract=on", "--cuda-host-only", "-x", "hip",
                    os.path.join(HERE, "geno_line.cpp"), "-o", exe], check=True, capture_output=True)
    r = json.loads(subprocess.run([exe], check=True, capture_output=True, text=True).stdout)
    assert r["differ"] == 0 and r["wrong"] == 0, r
    assert r["quick"] > r["total"] // 20 and r["quick"] < r["total"] and r["fired"] > 1000, r
