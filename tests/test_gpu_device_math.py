"""Reciprocal, square root, exp, erf and tanh as the FP64 solver writes them
out (GPU), against extended precision over the ranges they are used in.

Bounds in units of the last place of the result.  Reciprocal and square root:
the last Newton step rounds once, on a correction far below an ulp, so within
one.  exp(-x): the rounding of s + s m with m = expm1(r) right to an ulp and
|m| < 0.42, so within two; 1 - exp(-x) likewise (below x = 0.35 it is -m
itself).  erf / 2: Horner's last steps and the product round once each on terms
that do not cancel, so within two.  tanh = (1 - E) / (1 + E): three roundings on
top of exp's, so within four."""
import ctypes as C
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
LD = np.longdouble


@pytest.fixture(scope="module")
def lib():
    path = os.path.join(HERE, "libdevice_math.so")
    if not os.path.exists(path):
        from paper_2606_17772_amd import build
        build.build_test_kernels()
    # torch's HIP runtime first, as the package's own loader has it: a library
    # loaded before it would bind a second runtime, whose devices know nothing
    # of torch's arrays
    from paper_2606_17772_amd import _lib
    _lib.load()
    L = C.CDLL(path)
    L.device_math.argtypes = [C.c_int, C.c_void_p, C.c_void_p, C.c_int]
    return L


def _run(lib, op, x):
    import torch
    a = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    y = torch.empty_like(a)
    torch.cuda.synchronize()
    assert lib.device_math(op, a.data_ptr(), y.data_ptr(), a.numel()) == 0
    torch.cuda.synchronize()
    return y.cpu().numpy()


def _ulps(got, want):
    return float(np.max(np.abs(got.astype(LD) - want) / np.spacing(np.abs(want.astype(np.float64))).astype(LD)))


def _logs(lo, hi, n=200000, seed=0):
    return np.exp(np.random.default_rng(seed).uniform(np.log(lo), np.log(hi), n))


def _half_erf(z):
    """erf(z) / 2 for |z| <= 1: its power series."""
    z = z.astype(LD)
    term, s = z.copy(), z.copy()
    for n in range(1, 40):
        term = -term * z * z / n
        s = s + term / (2 * n + 1)
    return s / np.sqrt(LD(4) * np.arctan(LD(1)))


CASES = {
    "recip": (0, lambda: np.concatenate([_logs(1e-290, 1e290), 1 + np.random.default_rng(1).random(200000)]),
              lambda x: LD(1) / x.astype(LD), 1.0),
    "sqrt": (1, lambda: np.concatenate([_logs(1e-290, 1e290), 1 + 3 * np.random.default_rng(2).random(200000)]),
             lambda x: np.sqrt(x.astype(LD)), 1.0),
    "exp": (2, lambda: np.concatenate([_logs(1e-30, 700.0), np.linspace(0.0, 700.0, 100001)]),
            lambda x: np.exp(-x.astype(LD)), 2.0),
    "one_minus_exp": (3, lambda: np.concatenate([_logs(1e-300, 700.0), np.linspace(1e-3, 3.0, 100001)]),
                      lambda x: -np.expm1(-x.astype(LD)), 2.0),
    "half_erf": (4, lambda: np.concatenate([_logs(1e-30, 1.0), np.linspace(-1.0, 1.0, 100000)]), _half_erf, 2.0),
    "tanh": (5, lambda: np.concatenate([_logs(1e-30, 40.0), np.linspace(-25.0, 25.0, 100000)]),
             lambda x: np.tanh(x.astype(LD)), 4.0),
}


@pytest.mark.parametrize("name", CASES)
def test_within_its_units_of_the_last_place(lib, name):
    op, points, exact, bound = CASES[name]
    x = points()
    w = _ulps(_run(lib, op, x), exact(x))
    print(f"{name}: {w:.3f} ulp over {x.size} points")
    assert w <= bound


def test_ends_of_the_ranges(lib):
    inf, nan = np.inf, np.nan
    assert _run(lib, 2, np.array([0.0, 800.0, 1e300, inf])).tolist() == [1.0, 0.0, 0.0, 0.0]
    assert _run(lib, 3, np.array([0.0, 800.0, inf])).tolist() == [0.0, 1.0, 1.0]
    assert _run(lib, 5, np.array([0.0, 20.0, -20.0, 1e300])).tolist() == [0.0, 1.0, -1.0, 1.0]
    for op in range(6):
        assert np.isnan(_run(lib, op, np.array([nan]))).all()
    assert np.isnan(_run(lib, 1, np.array([-1.0]))).all()
