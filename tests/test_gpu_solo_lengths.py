"""First-order GPU parity of the single work-group solver at run-time lengths.

2D Ga plans whose complex double grid fits one work-group's LDS run whole CG
iterations in one work-group per solve, whatever their 3,5,7-smooth lengths.
Every solve stops after K steps and each entry of the bounds must match the
oracle's bounds of the same iterates to 1e-11 of the reference norm (Remark
CG: the iterate is a fixed polynomial in the operator), for grids from one
point along an axis to the largest that fit, with every radix first and last
in a schedule, remainders of the 256-, 512- and 1024-thread forms, and scalar,
anisotropic and matrix materials.  The FP32-iteration form must match the FP64
run of K32 steps at contrast 10 to 1e-7.  Solves of plans that share a grid
but not an order run in one batch and must give what they give alone.
"""

import numpy as np
import pytest

import synth
from oracle import ga, material

pytestmark = pytest.mark.gpu

K = 10
K32 = 2
# orders; double grids (5, 1) (1, 9) (5, 5) (9, 15) (21, 21) (25, 49) (27 is no double grid) ...
ORDERS = ((3, 1), (1, 5), (3, 3), (5, 7), (11, 11), (13, 25), (17, 23), (31, 33), (5, 41), (41, 5), (61, 3), (3, 365),
          (37, 37), (37, 61), (113, 11), (15, 73))
ORDERS32 = ((11, 11), (51, 51), (61, 53), (51, 63), (37, 87))


@pytest.fixture(scope="module")
def fg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1412_2033_amd import fftgal
    fftgal.load_library()
    return fftgal


def _micro(N, kind, contrast):
    if kind == "disc":
        return synth.random_circles(3, k_lo=4, k_hi=8, r_lo=0.05, r_hi=0.12, contrast=contrast)
    if kind == "poly":
        return synth.polycrystal(6, (21, 15), d=2, n_grains=7, log10_hi=np.log10(contrast))
    m = synth.cube_inclusion_aniso(0.45, 7, d=2)
    m["A_in"] = m["A_in"] * (contrast / 1000.0)
    return m


def _run(fg, micro, N, precision, k, solo=True, **kw):
    print("solo lengths N=%s %s k=%d %s" % (N, precision, k, kw), flush=True)
    plan = fg.Plan(2, N, precision, P=micro.get("P"), **kw)
    try:
        plan.set_timing(True)
        res = plan.run(micro, rtol=0.0, maxit=k)
        t = plan.read_timing()
        assert (t["solo"][1] > 0) == solo and (t["cg_update"][1] == 0) == solo, t
        return res
    finally:
        plan.close()


def _err(res, ref):
    return max(float(np.max(np.abs(res[k] - ref[k])) / np.linalg.norm(ref[k])) for k in ("upper", "lower"))


@pytest.mark.parametrize("N", ORDERS)
@pytest.mark.parametrize("kind", ("disc", "aniso", "poly"))
def test_truncated_matches_oracle(fg, N, kind):
    micro = _micro(N, kind, 50.0)
    res = _run(fg, micro, N, "fp64", K, tensor=kind == "poly")
    assert _err(res, ga.ga_bounds(material.make_material(micro), N, tol=0.0, maxit=K)) <= 1e-11


@pytest.mark.parametrize("N", ORDERS32)
def test_fp32_matches_fp64(fg, N):
    micro = _micro(N, "disc", 10.0)
    assert _err(_run(fg, micro, N, "fp32", K32), _run(fg, micro, N, "fp64", K32, solo=False, separate_passes=True)) <= 1e-7


def test_batch_of_orders_on_one_grid(fg):
    orders = ((15, 15), (17, 15), (17, 17))  # all on the 35 x 35 grid
    micro = _micro(None, "disc", 30.0)
    batch = fg.Batch(capacity=16)
    plans = [fg.Plan(2, N, "fp64", stream=batch.stream, concurrent=True) for N in orders]
    assert all(p.M == (35, 35) for p in plans)
    left = 0
    for p in plans:
        p.set_material(micro)
        for kind in (0, 1):
            for a in (0, 1):
                batch.add(p, kind, a, rtol=1e-9)
                left += 1
    while left:
        batch.step(16)
        left -= len(batch.poll())
    for p, N in zip(plans, orders):
        mixed = p.bounds()
        alone = fg.Plan(2, N, "fp64")
        ref = alone.run(micro, rtol=1e-9)
        assert np.array_equal(mixed[0], ref["upper"]) and np.array_equal(mixed[1], ref["lower"])
        alone.close()
        p.close()
    batch.close()
