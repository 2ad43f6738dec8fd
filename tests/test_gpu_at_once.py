"""GPU tests of the solves of one call that run at once.

A call for several solves runs them in shared launches, as many at once as the
plan's workspace holds: all 2d, the d of one kind, or one after another.  Each
solve keeps its own reductions, so iteration counts, residuals, the energies of
every iterate and the bounds must equal bitwise those of the solves made by one
call each (which always run alone).  The cases cover the single work-group
solver, the per-pass kernels, whole planes, FP32 checkpoints, both counts of
solves at once, GaNi plans (direct and Bluestein transforms), matrix images,
warm starts and the bound tolerance; every plan is also made without the room
(FFTGAL_ONE_AT_A_TIME) and with one buffer set per solve (FFTGAL_CONCURRENT).
"""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fg():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1412_2033_amd import fftgal
    fftgal.load_library()
    return fftgal


def _grf(N, contrast=30.0, gani=False):
    P = N if gani else tuple(2 * n - 1 for n in N)
    return synth.grf_voxels(11, P, d=len(N), corr_len=0.1, a_incl=contrast)


# name: (N, precision, rtol, maxit, solves at once, plan arguments, material)
CASES = {
    "solo": ((11, 11), "fp64", 1e-10, 500, 4, {}, lambda N: synth.square_inclusion(2, 0.6, 1.0, 10.0)),
    "solo_fp32": ((63, 41), "fp32", 1e-7, 500, 4, {}, lambda N: synth.random_circles(5)),
    "passes_fp32": ((63, 63), "fp32", 1e-7, 500, 4, {"separate_passes": True}, lambda N: synth.random_circles(5)),
    "tensor": ((95, 67), "fp64", 1e-8, 500, 4, {"tensor": True}, lambda N: synth.polycrystal(3, (39, 27), d=2)),
    "two_at_once": ((1013, 1013), "fp64", 1e-6, 500, 2, {}, lambda N: synth.circle_inclusion_vf(0.3, 1.0, 100.0)),
    "planes": ((21, 21, 21), "fp64", 1e-8, 500, 6, {}, _grf),
    "planes_fp32": ((9, 23, 21), "fp32", 5e-6, 500, 6, {}, _grf),
    "aniso_fp32": ((23, 23, 23), "fp32", 5e-6, 200, 6, {}, lambda N: synth.cube_inclusion_aniso(0.45, 4)),
    "three_at_once": ((63, 63, 63), "fp64", 1e-6, 500, 3, {}, lambda N: synth.cube_inclusion_aniso(0.45, 4)),
    "two_components": ((113, 113, 5), "fp64", 1e-8, 500, 3, {}, _grf),
    "stopped": ((21, 15, 9), "fp64", 0.0, 7, 6, {}, _grf),
    "no_iterations": ((95, 67), "fp64", 1e-8, 0, 4, {}, _grf),
    "gani_2d": ((33, 41), "fp64", 1e-8, 500, 4, {"scheme": "gani"}, lambda N: _grf(N, gani=True)),
    "gani_3d_fp32": ((21, 11, 9), "fp32", 5e-6, 500, 6, {"scheme": "gani"}, lambda N: _grf(N, gani=True)),
}


def _solves(d):
    return [(k, a) for k in (0, 1) for a in range(d)]


def _one_each(plan, rtol, maxit):
    return [(plan.solve_primal, plan.solve_dual)[k](a, rtol, maxit)[0][0] for k, a in _solves(plan.d)]


def _by_kind(plan, rtol, maxit):
    return plan.solve_primal(-1, rtol, maxit)[0] + plan.solve_dual(-1, rtol, maxit)[0]


def _all(fg):
    def run(plan, rtol, maxit):
        ip, idl, _ = fg.fftgal_solve_all(plan.handle, plan.d, rtol, maxit)
        return ip + idl
    return run


def _state(plan, solve, rtol, maxit):
    infos = solve(plan, rtol, maxit)
    return infos, [plan.history(k, a) for k, a in _solves(plan.d)], plan.bounds()[:2]


def _same(a, b):
    assert a[0] == b[0]
    for x, y in zip(a[1] + list(a[2]), b[1] + list(b[2])):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("name", sorted(CASES))
def test_equals_one_call_per_solve(fg, name):
    N, precision, rtol, maxit, at_once, kw, make = CASES[name]
    d = len(N)
    micro = make(N)
    print("at once: %s N=%s %s" % (name, N, precision), flush=True)
    kw = dict(kw, P=micro.get("P"))
    ref = None
    for how in ({}, {"at_once": False}, {"concurrent": True}):
        plan = fg.Plan(d, N, precision, **kw, **how)
        try:
            plan.set_material(micro)
            if ref is None:
                ref = _state(plan, _one_each, rtol, maxit)
                assert all(i["iters"] > 0 for i in ref[0]) == (maxit > 0)
            for solve in (_by_kind, _all(fg)):
                _same(_state(plan, solve, rtol, maxit), ref)
            # solves alone again after solves at once, on what those left behind
            _same(_state(plan, _one_each, rtol, maxit), ref)
        finally:
            plan.close()
    flags = fg.PRECISIONS[precision] | (fg.TENSOR if kw.get("tensor") else 0)
    scheme = kw.get("scheme", "ga")
    room = fg.fftgal_workspace_bytes(d, N, flags, scheme=scheme) - \
        fg.fftgal_workspace_bytes(d, N, flags | fg.ONE_AT_A_TIME, scheme=scheme)
    assert (room > 0) == (at_once > 1)


@pytest.mark.parametrize("N,coarse", (((45, 45), (21, 21)), ((21, 15, 15), (9, 9, 9))))
@pytest.mark.parametrize("precision", ("fp64", "fp32"))
@pytest.mark.parametrize("start", ("warm", "btol"))
def test_warm_starts_and_bound_tolerance(fg, N, coarse, precision, start):
    d = len(N)
    micro = synth.square_inclusion(d, 0.6, 1.0, 20.0)
    rtol = 1e-8 if precision == "fp64" else 5e-6
    print("at once: %s N=%s %s" % (start, N, precision), flush=True)
    pc = fg.Plan(d, coarse, precision)
    plan = fg.Plan(d, N, precision)
    try:
        pc.run(micro, rtol=rtol)
        states = []
        for solve in (_one_each, _by_kind, _all(fg)):
            plan.set_material(micro)
            if start == "warm":
                plan.warm_start(pc)
            else:
                plan.set_bound_tol(1e-4)
            states.append(_state(plan, solve, rtol, 500))
        for s in states[1:]:
            _same(s, states[0])
    finally:
        pc.close()
        plan.close()
