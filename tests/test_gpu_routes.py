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
