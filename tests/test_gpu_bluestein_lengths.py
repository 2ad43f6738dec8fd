"""First-order GPU parity of the compile-time Bluestein passes.

GaNi and reduced-Ga plans transform the orders themselves; an order that is
not 3,5,7-smooth runs as a circular convolution of the smallest odd smooth
length L >= 2 n - 1 (Bluestein's identity), in kernels compiled for each L.
GaNi solves (isotropic voxels) stop after K steps and each entry of both
matrices must match the oracle's of the same iterates to 1e-11 of the reference
norm, with n on every axis; so must the bounds of reduced plans.  The orders
reach the smallest and largest n of an L, tiles of one and of several pencils
and row pairs, and the longest L.  The FP32-iteration form must match FP64 after
K32 steps at contrast 10 to 1e-7.
"""

import numpy as np
import pytest

import synth
from oracle import gani, material, reduced

pytestmark = pytest.mark.gpu

K = 4
K32 = 2
ORDERS_3D = (11, 13, 17, 29, 41, 53, 61, 97, 99, 113, 121, 163, 187, 201)
ORDERS_2D = (11, 23, 43, 69, 87, 113, 123, 201, 257, 361, 421, 509, 605, 787, 857, 1013)


@pytest.fixture(scope="module")
def fg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1412_2033_amd import fftgal
    fftgal.load_library()
    return fftgal


def _run(fg, micro, N, precision, k, scheme):
    print("bluestein N=%s %s %s k=%d" % (N, scheme, precision, k), flush=True)
    plan = fg.Plan(len(N), N, precision, P=micro.get("P"), scheme=scheme)
    try:
        return plan.run(micro, rtol=0.0, maxit=k)
    finally:
        plan.close()


def _err(res, ref):
    return max(float(np.max(np.abs(res[k] - ref[k])) / np.linalg.norm(ref[k])) for k in ("upper", "lower"))


def _grids(n, d):
    out = []
    for axis in range(d):
        N = [5] * d
        N[axis] = n
        out.append(tuple(N))
    return out + ([(n, 11)] if d == 2 else [])


def _check(fg, n, d):
    for N in _grids(n, d):
        micro = synth.grf_voxels(11, N, d=d, corr_len=0.1, vf=0.4, a_matrix=1.0, a_incl=50.0)
        ref = gani.gani(micro, N, tol=0.0, maxit=K)
        res = _run(fg, micro, N, "fp64", K, "gani")
        assert _err(res, {"upper": ref["A_gani"], "lower": np.linalg.inv(ref["B_gani"])}) <= 1e-11
        easy = synth.grf_voxels(11, N, d=d, corr_len=0.1, vf=0.4, a_matrix=1.0, a_incl=10.0)
        assert _err(_run(fg, easy, N, "fp32", K32, "gani"), _run(fg, easy, N, "fp64", K32, "gani")) <= 1e-7


@pytest.mark.parametrize("n", ORDERS_2D)
def test_gani_2d(fg, n):
    _check(fg, n, 2)


@pytest.mark.parametrize("n", ORDERS_3D)
def test_gani_3d(fg, n):
    _check(fg, n, 3)


@pytest.mark.parametrize("N", ((11, 13), (61, 5), (5, 113), (11, 5, 13), (5, 41, 3)))
def test_reduced(fg, N):
    micro = synth.grf_voxels(11, tuple(2 * n - 1 for n in N), d=len(N), corr_len=0.1, vf=0.4, a_matrix=1.0, a_incl=50.0)
    ref = reduced.reduced_bounds(material.make_material(micro), N, tol=0.0, maxit=K)
    assert _err(_run(fg, micro, N, "fp64", K, "reduced"), ref) <= 1e-11
