"""A step that stops (GPU): whatever launches carry it, it names a node next to
the one whose value spoils it and leaves the state as it was.

The update kernels whose waves share LDS read the stop flag once per block:
the flag may be set by another block of the same launch while a block starts."""
import re

import numpy as np
import pytest

import workloads as WL
from tests.helpers import gpu_params, settings

pytestmark = pytest.mark.gpu

REACH = 8  # a node's new value depends on nodes at most this far (two sweeps and two assemblies)


def _node(text):
    return [int(v) for v in re.search(r"grid (\d+) node \((-?\d+), (-?\d+)\)", text).groups()]


@pytest.mark.parametrize("launches", ["joined", "separate", "fused", "node_fusion"])
@pytest.mark.parametrize("bad", [(20, 5), (130, 199)])
def test_stop_names_a_bad_node(launches, bad):
    from paper_2606_17772_amd import FdcgksError, Problem
    nx, ny = 200, 140
    pr = WL.random_smooth2d(nx, ny, seed=4)
    P, D = pr.P.copy(), pr.D.copy()
    P[3, bad[0], bad[1]] = -10.0
    pb = Problem(gpu_params(settings(dim=2, nx=nx, ny=ny, lx=1.0)))
    pb.set_state_stacked(0, P)
    pb.set_state_stacked(1, D)
    pb.fuse_stage = launches == "fused"
    if launches == "separate":
        pb.set_tile("edge", 64, 2)
    pb.fuse_nodes = launches == "node_fusion"
    with pytest.raises(FdcgksError) as ei:
        pb.step(nsteps=3, dt=1e-4)
    grid, i, j = _node(str(ei.value))
    assert grid in (0, 1)
    near = [min((a - b) % n, (b - a) % n) for a, b, n in ((i, bad[1], nx), (j, bad[0], ny))]
    assert max(near) <= REACH, (i, j)
    assert np.array_equal(pb.get_state_stacked(0), P) and np.array_equal(pb.get_state_stacked(1), D)


@pytest.mark.parametrize("mode", ["graph", "phased", "persistent"])
def test_batch_stop_names_a_bad_node(mode):
    from paper_2606_17772_amd import Batch, FdcgksError
    sizes = [(40, 33), (70, 65), (24, 130)]
    cases = [WL.random_smooth2d(nx, ny, seed=5 + m) for m, (nx, ny) in enumerate(sizes)]
    b = Batch([gpu_params(settings(dim=2, nx=nx, ny=ny, lx=1.0)) for nx, ny in sizes])
    b.set_mode(mode)
    states = [(c.P.copy(), c.D.copy()) for c in cases]
    states[1][1][0, 31, 66] = -1.0
    for m, st in enumerate(states):
        for g in (0, 1):
            b.set_state_stacked(m, g, st[g])
    with pytest.raises(FdcgksError) as ei:
        b.step(nsteps=3, cfl=0.3)
    m, i, j = [int(v) for v in re.search(r"member (\d+).*node \((-?\d+), (-?\d+)\)", str(ei.value)).groups()]
    nx, ny = sizes[m]
    assert m == 1
    assert max(min((a - c) % n, (c - a) % n) for a, c, n in ((i, 66, nx), (j, 31, ny))) <= REACH
    for m, st in enumerate(states):
        for g in (0, 1):
            assert np.array_equal(b.get_state_stacked(m, g), st[g])
