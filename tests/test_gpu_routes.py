"""Which launches carry a call (GPU), read from the per-kernel times: the
separate interface sweep, the joined sweeps (no node slot) or the fused stage
(no interface slot)."""
import numpy as np
import pytest

from tests.helpers import gpu_params, settings

pytestmark = pytest.mark.gpu


def _uniform(nx, ny, **kw):
    from paper_2606_17772_amd import Problem
    pb = Problem(gpu_params(settings(dim=2, nx=nx, ny=ny, lx=1.0, **kw)))
    S = np.zeros((12, ny, nx))
    S[0], S[3] = 1.0, 2.5
    for g in (0, 1):
        pb.set_state_stacked(g, S)
    return pb


def _route(pb):
    _, _, ms = pb.step_timed(nsteps=1, dt=1e-6)
    if ms["edge1"] == 0.0:
        return "fused"
    return "joined" if ms["node1"] == 0.0 else "separate"


@pytest.mark.parametrize("recon", ["conservative", "characteristic"])
@pytest.mark.parametrize("n,fp32,route", [(900, False, "fused"), (900, True, "joined"), (1460, True, "fused")])
def test_fused_stage_by_precision(n, fp32, route, recon):
    """FP32 fluxes want row chunks three times as tall (800^2: 0.88 fused
    against 0.75 ms unfused; FP64 0.70 against 0.75)."""
    assert _route(_uniform(n, n, fp32_flux=fp32, recon_vars=recon)) == route


def test_autotune_decides_the_launches():
    """A chosen shape selects a launch per kernel; autotune times that against
    the joined launches and keeps the faster, whatever was chosen before (at
    96 x 48 the joined ones: 41 against 73 us a step).  The shapes it reports
    give the same results when set."""
    import workloads as WL
    pr = WL.random_smooth2d(96, 48, seed=3)

    def make():
        pb = _uniform(96, 48)
        for g, S in ((0, pr.P), (1, pr.D)):
            pb.set_state_stacked(g, S)
        return pb

    a, b, c = make(), make(), make()
    assert _route(a) == "joined"
    for g, S in ((0, pr.P), (1, pr.D)):
        a.set_state_stacked(g, S)
    a.set_tile("update", 32, 4)
    tiles = a.autotune(reps=5)
    for kernel, (x, y) in tiles.items():
        b.set_tile(kernel, x, y)
    assert a.tiles() == b.tiles() == tiles
    for pb in (a, b, c):
        assert pb.step(nsteps=3, cfl=0.4)[1] == 3
    assert np.array_equal(a.get_state_all(), c.get_state_all()) and np.array_equal(b.get_state_all(), c.get_state_all())
    assert _route(b) == "separate" and _route(a) == "joined"


def _pinned(shape):
    import torch
    return torch.zeros(shape, dtype=torch.float64, pin_memory=True)


def test_pinned_arrays_as_device_pointers():
    """Memory that a kernel of the library does not take directly, handed over
    as a device pointer, goes through the runtime's copies: states of a problem
    and a batch in and out, and the adjoint's arrays, equal to the kernel route
    bit for bit."""
    import ctypes as C

    import torch

    import workloads as WL
    from paper_2606_17772_amd import Batch, Problem, _lib
    L = _lib.load()
    nx, ny = 37, 21
    pr = WL.random_smooth2d(nx, ny, seed=8)
    prm = gpu_params(settings(dim=2, nx=nx, ny=ny, lx=1.0))
    pb, b = Problem(prm), Batch([prm])

    def ptrs(t):
        return [C.c_void_p(t.data_ptr() + 8 * 4 * q * ny * nx) for q in range(3)]

    src, dst = _pinned((12, ny, nx)), _pinned((12, ny, nx))
    for g, S in ((0, pr.P), (1, pr.D)):
        src.copy_(torch.from_numpy(S))
        assert L.fdcgks_set_state(pb._h, g, *ptrs(src), 0, 1) == 0
        assert L.fdcgks_batch_set_state(b._h, 0, g, *ptrs(src), 1) == 0
        torch.cuda.synchronize()
        assert np.array_equal(pb.get_state_stacked(g), S) and np.array_equal(b.get_state_stacked(0, g), S)
        for call in (lambda: L.fdcgks_get_state(pb._h, g, *ptrs(dst), 0, 1),
                     lambda: L.fdcgks_batch_get_state(b._h, 0, g, *ptrs(dst), 1)):
            dst.zero_()
            assert call() == 0
            torch.cuda.synchronize()
            assert np.array_equal(dst.numpy(), S)
    lam = torch.from_numpy(np.random.default_rng(2).standard_normal((2, 12, ny, nx)))
    lin, lout = _pinned(lam.shape), _pinned(lam.shape)
    lin.copy_(lam)
    assert L.fdcgks_step_vjp(pb._h, C.c_double(1e-3), C.c_void_p(lin.data_ptr()), C.c_void_p(lout.data_ptr()), 1) == 0
    torch.cuda.synchronize()
    want = pb.step_vjp(1e-3, lam.numpy())
    # the reverse sweeps add by atomics: repeated calls differ by round-off (see test_gpu_adjoint's device arrays)
    assert np.abs(lout.numpy() - want).max() <= 1e-12 * np.abs(want).max()
