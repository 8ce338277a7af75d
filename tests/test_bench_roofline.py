"""The constants that bench.py reckons achieved rates from, and the launch it
attributes them to (CPU)."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def _row(kernel):
    """Counter row of a kernel as the code is now: cells of its table line (one
    marked "before" holds an earlier form's count)."""
    txt = open(os.path.join(ROOT, "profiles", "k_edges2d_shear2048.md")).read()
    rows = [ln for ln in txt.splitlines() if ln.startswith(f"| `{kernel}`") and ln.count("|") >= 8]
    now = [r for r in rows if "before" not in r.split("|")[1]]
    assert len(now) == 1, rows
    return [c.strip() for c in now[0].strip().strip("|").split("|")]


def test_constants_are_those_of_the_kernels_that_run():
    import bench
    edges = _row("k_edges2d<1, double, false>")
    assert bench.FLOPS_EXECUTED_PER_IFACE_POINT_STAGE1 == int(edges[4])
    assert abs(bench.TRAFFIC_BYTES_PER_LAUNCH_STAGE1 - (float(edges[5]) + float(edges[6])) * 1e9) <= 2e6
    assert bench.FLOPS_PER_NODE_SWEEP_STAGE1 == int(_row("k_nodes2d<1, double, false>")[4])


@pytest.mark.parametrize("stage,kms,kernel,flops", [
    ("fused", dict(edge1=0.0, node1=1.0, update1=4.0), "k_fused2d", 4415 * 2 * 100 ** 2),
    ("separate", dict(edge1=4.0, node1=1.0, update1=3.0), "k_edges2d", 3789 * 2 * 103 ** 2),
    # the joined sweeps' launch is in the interface slot and does the nodes too
    ("joined", dict(edge1=4.0, node1=0.0, update1=3.0), "k_sweeps2d", 3789 * 2 * 103 ** 2 + 499 * 2 * 102 ** 2)])
def test_rate_of_the_launch_that_ran(stage, kms, kernel, flops):
    import bench
    got, roof = bench.stage_roofline(kms, 2, 100)
    assert got == stage and roof["kernel"].startswith(kernel)
    assert roof["avg_launch_ms"] == 2.0
    assert roof["achieved"] == round(flops / 2e-3 / 1e12, 3)
    assert (roof["traffic"] is None) == (stage == "joined")


def test_tiles_are_chosen_only_when_asked_for(monkeypatch):
    """Setting a shape selects a launch per kernel, so the default run sets none."""
    import bench
    monkeypatch.setattr(sys, "argv", ["bench.py"])
    assert bench.parse_tiles(bench.parse().tiles) == {}
    assert bench.parse_tiles(bench.DEFAULT_TILES) == {"edge": (64, 2), "node": (64, 1), "update": (128, 1)}


def test_executed_count_against_the_source(tmp_path):
    """The counted flop per interface point against the operations of the
    source it is compiled from (the solver in primitive slopes; test_opcount.py
    counts the form from moment vectors, which the FP32-flux variant runs).  The
    compiler folds and shares some of them (a fifth at most), and writes out
    exp (about 45 flop), erf (30), the reciprocal (10) and the square root (16)
    that the source count takes as one each."""
    import json
    import shutil
    import subprocess

    import bench
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "opcount")
    subprocess.run([hipcc, "-std=c++17", "-O1", "--cuda-host-only", "-x", "hip",
                    os.path.join(ROOT, "tests", "opcount_slopes.cpp"), "-o", exe], check=True, capture_output=True)
    c = json.loads(subprocess.run([exe], check=True, capture_output=True, text=True).stdout)
    assert (c["erfc"], c["exp"], c["sqrt"], c["div"]) == (4, 6, 4, 18), c
    written_out = 45 * c["exp"] + 30 * c["erfc"] + 10 * c["div"] + 16 * c["sqrt"]
    assert 0.8 * c["arith"] < bench.FLOPS_EXECUTED_PER_IFACE_POINT_STAGE1 < c["arith"] + written_out, c
