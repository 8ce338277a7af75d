"""State arrays in and out (CPU, the HIP runtime stood in for by
tests/state_io_host.cpp): a kernel runs on the problem's own device, whatever
device is current, and only on memory it reaches there; everything else goes
through the runtime's copies."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2606_17772_amd", "libfdcgks.so")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
EHIP = -3


@pytest.fixture(scope="module")
def calls(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("state_io") / "state_io")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "--cuda-host-only", "-x", "hip", os.path.join(HERE, "state_io_host.cpp"),
                    "-o", exe, "-rdynamic", "-ldl"], check=True, capture_output=True)
    out = subprocess.run([exe, LIB], check=True, capture_output=True, text=True).stdout
    rows = [ln.split("|") for ln in out.splitlines()]
    return {r[0]: dict(status=int(r[1]), current=int(r[2]), launches=r[3].split(), copies=int(r[4])) for r in rows}


@pytest.mark.parametrize("current", [0, 1])
@pytest.mark.parametrize("call", ["set", "get", "batch_set", "batch_get"])
def test_kernels_run_on_the_problems_device(calls, call, current):
    tail = "_other" if current else ""
    for where in ("host", "mine"):
        c = calls[f"{call}_{where}{tail}"]
        assert c["status"] == 0 and c["current"] == current
        assert len(c["launches"]) == 1 and "k_state_io" in c["launches"][0] and c["launches"][0].endswith("@0"), c
        assert c["copies"] == 0
    for where in ("peer", "pinned"):
        c = calls[f"{call}_{where}{tail}"]
        assert c["status"] == 0 and c["current"] == current
        assert c["launches"] == [] and c["copies"] == 12, c


@pytest.mark.parametrize("e", [59, 60, 61, 62])
def test_row_strides_beyond_the_address_space(calls, e):
    """2^e doubles a row: their bytes, or the arrays', do not fit 64 bits.  No
    kernel runs; the copies refuse a pitch below the row length."""
    c = calls[f"get_stride{e}"]
    assert c["launches"] == []
    if e >= 61:
        assert c["status"] == EHIP and c["copies"] == 0
