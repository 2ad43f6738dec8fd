"""First-order GPU parity of every transform length with compile-time kernels.

Each odd 3,5,7-smooth length n from 9 to 2025 has its own strided-axis, row
and energy kernels, with its own tiles, radix schedule and remainders.  As in
the truncated-iteration tests of the first six lengths (Remark CG: after k
steps the iterate is a fixed polynomial in the operator), every solve stops
after K steps and each entry of the bounds must match the oracle's bounds of
the same iterates to 1e-11 of the reference norm, with n on every axis in
turn: isotropic voxels (the isotropic row pass; odd row counts leave the last
pair of rows half empty) and an anisotropic inclusion (the general row pass).
The FP32-iteration form must match the FP64 run of K32 steps at contrast 10 to
1e-7.  The orders are the largest with 2 N - 1 <= n, so that the rows hold the
most points a Ga plan can have.  GaNi plans of order n transform rows of full
length and must match the oracle's matrices of the same iterates; those of
orders with factors 11 and 13 run lengths no double grid takes.
"""

import numpy as np
import pytest

import synth
from oracle import ga, gani, material

pytestmark = pytest.mark.gpu

K = 4
K32 = 2
LENGTHS = (9, 15, 21, 25, 35, 45, 49, 63, 75, 105, 135, 147, 175, 189, 243, 315, 343, 375, 405, 441, 525, 567,
           625, 675, 735, 875, 945, 1029, 1125, 1215, 1225, 1323, 1575, 1701, 1715, 1875)
# orders with factors 11 and 13, which GaNi and reduced plans transform directly
LENGTHS_13 = (11, 13, 33, 39, 55, 65, 77, 91, 99, 117, 121, 143, 165, 169, 195, 231, 273, 297, 325, 385)
LENGTHS_3D = tuple(n for n in LENGTHS if n <= 405)


@pytest.fixture(scope="module")
def fg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1412_2033_amd import fftgal
    fftgal.load_library()
    return fftgal


def _order(n):
    N = (n + 1) // 2
    return N if N % 2 else N - 1


def _axis(v, axis, d, other=5):
    N = [other] * d
    N[axis] = v
    return tuple(N)


def _micro(N, kind, contrast, P=None):
    d = len(N)
    if kind == "aniso":
        m = synth.cube_inclusion_aniso(0.45, 7 + d, d=d)
        m["A_in"] = m["A_in"] * (contrast / 1000.0)
        return m
    return synth.grf_voxels(11, P or tuple(2 * n - 1 for n in N), d=d, corr_len=0.1, vf=0.4, a_matrix=1.0,
                            a_incl=contrast)


def _err(res, ref):
    return max(float(np.max(np.abs(res[k] - ref[k])) / np.linalg.norm(ref[k])) for k in ("upper", "lower"))


def _run(fg, micro, N, precision, k, n, axis, **kw):
    print("length %d axis %d N=%s %s k=%d" % (n, axis, N, precision, k), flush=True)
    plan = fg.Plan(len(N), N, precision, P=micro.get("P"), separate_passes=True, **kw)
    try:
        assert plan.M[axis] == n
        return plan.run(micro, rtol=0.0, maxit=k)
    finally:
        plan.close()


def _check(fg, n, d, kind):
    for axis in range(d):
        N = _axis(_order(n), axis, d)
        micro = _micro(N, kind, 50.0)
        res = _run(fg, micro, N, "fp64", K, n, axis)
        assert _err(res, ga.ga_bounds(material.make_material(micro), N, tol=0.0, maxit=K)) <= 1e-11
        easy = _micro(N, kind, 10.0)
        assert _err(_run(fg, easy, N, "fp32", K32, n, axis), _run(fg, easy, N, "fp64", K32, n, axis)) <= 1e-7


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("kind", ("voxels", "aniso"))
def test_length_2d(fg, n, kind):
    _check(fg, n, 2, kind)


@pytest.mark.parametrize("n", LENGTHS_3D)
@pytest.mark.parametrize("kind", ("voxels", "aniso"))
def test_length_3d(fg, n, kind):
    _check(fg, n, 3, kind)


@pytest.mark.parametrize("n", (9, 27, 49, 75, 147, 315, 735) + LENGTHS_13)
def test_full_rows(fg, n):
    grids = [(5, n), (n, 5)] + ([(n, 5, 3), (5, n, 3), (3, 5, n)] if n <= 231 else [])
    for N in grids:
        micro = _micro(N, "voxels", 50.0, P=N)
        res = _run(fg, micro, N, "fp64", K, n, N.index(n), scheme="gani")
        ref = gani.gani(micro, N, tol=0.0, maxit=K)
        assert _err(res, {"upper": ref["A_gani"], "lower": np.linalg.inv(ref["B_gani"])}) <= 1e-11
        easy = _micro(N, "voxels", 10.0, P=N)
        assert _err(_run(fg, easy, N, "fp32", K32, n, N.index(n), scheme="gani"),
                    _run(fg, easy, N, "fp64", K32, n, N.index(n), scheme="gani")) <= 1e-7
