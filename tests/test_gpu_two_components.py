"""First-order GPU parity of the two-component passes of 3D gradient fields.

On 3D grids of at least 343,000 points the primal solves carry two components
instead of three between axis 1 and axis 2: the axis-1 passes have tiles of
their own for every length, and the axis-2 passes make three components of two
and two of three.  Each length with compile-time kernels is put on axis 1 and,
with another partner, on axis 2 of a grid that just exceeds the threshold; GaNi
plans do the same with the orders that are transformed directly (full rows) and
with orders that are transformed by Bluestein convolutions, the smallest and the
largest of every convolution length.

A primal solve stops after K steps.  The decrease of the energy in each step,
alpha_k (r_k, r_k), depends on the operator to first order and must match the
oracle's to 1e-11 of the initial energy.  The bounds of the FP32-iteration form
must match those of FP64 after K32 steps at contrast 10 to 1e-7.
"""

import numpy as np
import pytest

import synth
from oracle import ga, gani, material

pytestmark = pytest.mark.gpu

K = 4
K32 = 2
LEAST = 343000
LENGTHS = (9, 15, 21, 25, 35, 45, 49, 63, 75, 81, 105, 125, 135, 147, 175, 189, 225, 243, 245, 315, 343, 375,
           405, 729, 2025)
# orders with factors 11 and 13 that are transformed directly
# (which only GaNi and reduced plans transform)
DIRECT_13 = (11, 13, 33, 39, 55, 65, 77, 91, 99, 117, 121, 143, 165, 169, 195, 231, 273, 297, 325, 385)


@pytest.fixture(scope="module")
def fg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1412_2033_amd import fftgal
    fftgal.load_library()
    return fftgal


def _smooth(n):
    for p in (3, 5, 7):
        while n % p == 0:
            n //= p
    return n == 1


def _smooth_at_least(m):
    return next(n for n in range(m | 1, 4 * m + 9, 2) if _smooth(n))


def _bluestein_orders():
    ends = {}
    for n in range(11, 204, 2):
        L = _smooth_at_least(2 * n - 1)
        if not _smooth(n) and n not in DIRECT_13 and L <= 405:
            ends.setdefault(L, []).append(n)
    return sorted({n for v in ends.values() for n in (v[0], v[-1])})


def _grid(n, partner, fill):
    need = LEAST / (n * partner)
    return n, partner, next((m for m in fill if m >= need), fill[-1])


def _order(n):
    N = (n + 1) // 2
    return N if N % 2 else N - 1


def _voxels(contrast):
    return synth.grf_voxels(11, (15, 13, 9), d=3, corr_len=0.15, vf=0.4, a_matrix=1.0, a_incl=contrast)


def _check(fg, N, M, scheme):
    a = sum(N) // 2 % 3
    micro = _voxels(50.0)
    print("two components %s N=%s M=%s alpha=%d" % (scheme, N, M, a), flush=True)
    plan = fg.Plan(3, N, "fp64", P=micro["P"], scheme=scheme)
    try:
        assert plan.M == M and np.prod(M) >= LEAST
        plan.set_material(micro)
        plan.solve_primal(a, 0.0, K)
        got = plan.history(0, a)
    finally:
        plan.close()
    E = np.eye(3)[a]
    if scheme == "gani":
        AM = gani.sample(micro, N, "A")
    else:
        AM = material.double_grid_matrix(material.make_material(micro), N, tuple(2 * n - 1 for n in N), "A")
    _, info = ga.solve(AM, N, E, "E", 0.0, K)
    steps = np.array(info["alphas"]) * np.array(info["rr"][:K])
    assert len(got) == K + 1 and np.min(steps) > 1e-6 * got[0]
    assert np.max(np.abs(got[:-1] - got[1:] - steps)) <= 1e-11 * got[0]
    easy = _voxels(10.0)
    res = {}
    for precision in ("fp64", "fp32"):
        plan = fg.Plan(3, N, precision, P=easy["P"], scheme=scheme)
        try:
            res[precision] = plan.run(easy, rtol=0.0, maxit=K32)
        finally:
            plan.close()
    for key in ("upper", "lower"):
        ref = res["fp64"][key]
        assert np.max(np.abs(res["fp32"][key] - ref)) <= 1e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("k", range(len(LENGTHS)))
def test_lengths(fg, k):
    M = _grid(LENGTHS[k], LENGTHS[-1 - k], LENGTHS)
    N = tuple(_order(m) for m in M)
    assert tuple(_smooth_at_least(2 * n - 1) for n in N) == M
    _check(fg, N, M, "ga")


def _direct_orders():
    return sorted(DIRECT_13 + tuple(n for n in LENGTHS + (27,) if n <= 405))


@pytest.mark.parametrize("k", range(len(_direct_orders())))
def test_direct_orders(fg, k):
    orders = _direct_orders()
    N = _grid(orders[k], orders[-1 - k], orders)
    _check(fg, N, N, "gani")


@pytest.mark.parametrize("k", range(len(_bluestein_orders())))
def test_bluestein_orders(fg, k):
    orders = _bluestein_orders()
    N = _grid(orders[k], orders[-1 - k], tuple(range(9, 4001, 2)))
    _check(fg, N, N, "gani")
