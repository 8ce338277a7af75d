"""Whole 1D runs in LDS (up to 512 nodes in all) and through memory (more):
bit for bit the single stages of the same problem, at the edges of the two
kernels' ranges; the stops at t_end and at a non-physical state (GPU)."""
import numpy as np
import pytest

import workloads as WL
from tests.helpers import TOL, gpu_params, oracle_par, relerr, settings
from tests.test_gpu_parity1d import _floors, _gpu_state, _problem, _rough1d

pytestmark = pytest.mark.gpu

# nodes per line, lines, the rest: the smallest line (ghosts on both sides of
# one node), partial and full waves, the last sizes in LDS, the first beyond
CASES = [
    (4, 1, {}), (5, 2, {"flux_order": 8}), (61, 1, {"bc": "reflecting"}), (64, 2, {"bc": "zero_gradient"}),
    (255, 2, {"bc": "reflecting", "flux_order": 8}), (256, 2, {}), (257, 2, {}), (512, 1, {"bc": "zero_gradient"}),
    (513, 1, {}), (300, 1, {"recon_vars": "characteristic"}), (129, 1, {"mu": 1e-3, "prandtl": 0.72, "grad_carried": 1}),
    (200, 1, {"variant": "linear"}),
]


def _case(n, lines, kw):
    s = settings(dim=1, nx=n, lx=1.0, dual_1d=int(lines == 2), **kw)
    return s, np.concatenate([_rough1d(n, 5 + q) for q in range(lines)])


@pytest.mark.parametrize("n,lines,kw", CASES)
def test_run_is_its_stages_bit_for_bit(oracle, n, lines, kw):
    s, S = _case(n, lines, kw)
    dt = 0.1 / n
    pb = _problem(s, S)
    pb.debug_stage(1, dt)
    one = pb.debug_stage(2, dt).reshape(S.shape)
    t, k = pb.step(nsteps=1, dt=dt)
    assert k == 1
    got = _gpu_state(pb, lines)
    assert np.array_equal(got, one)
    o1, a1 = oracle.stage1d(oracle_par(oracle, s), 1, dt, S)
    o2 = oracle.stage1d(oracle_par(oracle, s), 2, dt, o1, a1)
    err, where = relerr(got, o2, _floors(S, L=1.0), ndim_plane=1)
    assert err <= TOL, (where, err)


@pytest.mark.parametrize("n", [100, 600])
def test_cfl_run_in_one_call_and_step_by_step(n):
    S = WL.advection1d(n, noise=0.0).S
    s = settings(dim=1, nx=n, lx=2.0, dual_1d=1)
    a, b = _problem(s, S), _problem(s, S)
    t, k = a.step(nsteps=7, cfl=0.5)
    tb = 0.0
    for _ in range(7):
        tb, kb = b.step(nsteps=1, cfl=0.5, t=tb)
        assert kb == 1
    assert k == 7 and t == tb and np.array_equal(_gpu_state(a, 2), _gpu_state(b, 2))
    # a step clipped at t_end, and none beyond it
    t2, k2 = a.step(nsteps=5, cfl=0.5, t=t, t_end=t + 1e-6)
    assert k2 == 1 and t2 == t + 1e-6
    before = _gpu_state(a, 2)
    t3, k3 = a.step(nsteps=5, cfl=0.5, t=t2, t_end=t2)
    assert k3 == 0 and t3 == t2 and np.array_equal(before, _gpu_state(a, 2))


@pytest.mark.parametrize("n", [100, 600])
def test_failing_step_leaves_the_last_good_state(n):
    from paper_2606_17772_amd import FdcgksError
    S = WL.advection1d(n, noise=0.0, dual=False).S
    pb = _problem(settings(dim=1, nx=n, lx=2.0), S)
    pb.step(nsteps=1, cfl=0.5)
    good = _gpu_state(pb, 1)
    with pytest.raises(FdcgksError):
        pb.step(nsteps=3, dt=50.0 / n)  # far beyond any stable step
    assert np.isfinite(_gpu_state(pb, 1)).all()
    pb2 = _problem(settings(dim=1, nx=n, lx=2.0), S)
    pb2.step(nsteps=1, cfl=0.5)
    bad = good.copy()
    bad[0, 2, n // 2] = -1.0  # negative energy: the first stage fails, nothing moves
    pb2.set_state_stacked(0, bad[0])
    with pytest.raises(FdcgksError):
        pb2.step(nsteps=2, cfl=0.5)
    assert np.array_equal(_gpu_state(pb2, 1), bad)
