"""First-order GPU parity of the whole-plane passes of small 3D grids.

3D Ga plans with isotropic materials and equal double grids of n <= 63 points
along axes 2 and 3 transform each plane x1 in one pass between the axis-1
passes.  Every solve stops after K steps and each entry of the bounds must
match the oracle's bounds of the same iterates to 1e-11 of the reference norm
(the FP32-iteration form the FP64 run of K32 steps at contrast 10 to 1e-7), for
every such length, with orders that fill the half spectra of axes 2 and 3 and
with smaller, unequal ones.  Unequal grids and anisotropic materials keep the
axis-2 and row passes.
"""

import numpy as np
import pytest

import synth
from oracle import ga, material

pytestmark = pytest.mark.gpu

K = 4
K32 = 2
LENGTHS = (9, 15, 21, 25, 35, 45, 49, 63)


@pytest.fixture(scope="module")
def fg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1412_2033_amd import fftgal
    fftgal.load_library()
    return fftgal


def _orders(n):
    N = (n + 1) // 2
    N -= 1 - N % 2
    return (3, N, N), (7, N, N - 2 if N > 9 else N), (5, N - 2 if N > 9 else N, N)


def _voxels(N, contrast):
    return synth.grf_voxels(11, tuple(2 * m - 1 for m in N), d=3, corr_len=0.1, vf=0.4, a_matrix=1.0, a_incl=contrast)


def _run(fg, micro, N, precision, k, iso=True):
    print("N=%s %s k=%d" % (N, precision, k), flush=True)
    plan = fg.Plan(3, N, precision, P=micro.get("P"))
    try:
        planes = iso and plan.M[1] == plan.M[2] <= 63
        plan.set_material(micro)
        plan.set_timing(True)
        plan.read_timing()
        plan.solve_primal(0, 0.0, k)
        plan.solve_dual(0, 0.0, k)
        t = plan.read_timing()
        assert t["row"][1] >= 2 * k
        assert (t["pencil_inv"][1] == 0) == planes
        plan.set_timing(False)
        return plan.run(micro, rtol=0.0, maxit=k)
    finally:
        plan.close()


def _err(res, ref):
    return max(float(np.max(np.abs(res[k] - ref[k])) / np.linalg.norm(ref[k])) for k in ("upper", "lower"))


@pytest.mark.parametrize("n", LENGTHS)
def test_planes(fg, n):
    for N in _orders(n):
        micro = _voxels(N, 50.0)
        res = _run(fg, micro, N, "fp64", K)
        assert _err(res, ga.ga_bounds(material.make_material(micro), N, tol=0.0, maxit=K)) <= 1e-11
        easy = _voxels(N, 10.0)
        assert _err(_run(fg, easy, N, "fp32", K32), _run(fg, easy, N, "fp64", K32)) <= 1e-7


def test_other_materials_and_grids_keep_the_passes(fg):
    aniso = synth.cube_inclusion_aniso(0.45, 10, d=3)
    aniso["A_in"] = aniso["A_in"] * 0.05
    N = (5, 11, 11)
    res = _run(fg, aniso, N, "fp64", K, iso=False)
    assert _err(res, ga.ga_bounds(material.make_material(aniso), N, tol=0.0, maxit=K)) <= 1e-11
    N = (5, 11, 7)
    micro = _voxels(N, 50.0)
    res = _run(fg, micro, N, "fp64", K)  # double grids of 21 and 15 points
    assert _err(res, ga.ga_bounds(material.make_material(micro), N, tol=0.0, maxit=K)) <= 1e-11
