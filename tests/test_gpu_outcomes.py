"""GPU tests of the outcomes a run of all solves reports.

Plan.run solves both sides in one call.  A breakdown of the conjugate gradients
on one side must be raised whatever the outcome of the other, as the call for
that side alone raises it.  Conductivities near 1e104 and 1e-104 give one: the
sums (p, K p) grow with the cube of the material's scale, so those of the side
with the large material overflow, while those of the other stay finite (and
that side stops at its iteration limit).
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


def _scaled(scale):
    return synth.square_inclusion(2, 0.6, scale, 10.0 * scale)


@pytest.mark.parametrize("separate", (False, True))
@pytest.mark.parametrize("side", (0, 1))
def test_breakdown_of_one_side_is_raised(fg, side, separate):
    # the side of the large material breaks down
    scale = (1e104, 1e-104)[side]
    N = (11, 11)
    print("breakdown side %d separate %s" % (side, separate), flush=True)
    plan = fg.Plan(2, N, "fp64", separate_passes=separate)
    try:
        plan.set_material(_scaled(scale))
        solve = (plan.solve_primal, plan.solve_dual)
        with pytest.raises(fg.FftgalError) as e:
            solve[side](-1, 1e-10, 2)
        assert e.value.code == -6
        assert solve[1 - side](-1, 1e-10, 2)[1] == -4
        assert fg.fftgal_outcome(plan.handle, 1 - side) == -4
        with pytest.raises(fg.FftgalError) as e:
            plan.run(_scaled(scale), rtol=1e-10, maxit=2)
        assert e.value.code == -6 and "breakdown" in str(e.value)
    finally:
        plan.close()


def test_sides_report_their_own_outcome(fg):
    plan = fg.Plan(2, (11, 11), "fp64")
    try:
        micro = _scaled(1.0)
        with pytest.raises(fg.FftgalError) as e:
            fg.fftgal_outcome(plan.handle, 0)  # nothing solved yet
        assert e.value.code == -5
        res = plan.run(micro, rtol=1e-10, maxit=2)
        assert (res["status_primal"], res["status_dual"]) == (-4, -4)
        res = plan.run(micro, rtol=1e-10)
        assert (res["status_primal"], res["status_dual"]) == (0, 0)
        iters = [max(i["iters"] for i in res["info_" + s]) for s in ("primal", "dual")]
        if iters[0] != iters[1]:
            maxit = min(iters)
            res = plan.run(micro, rtol=1e-10, maxit=maxit)
            assert [res["status_primal"], res["status_dual"]] == [0 if i <= maxit else -4 for i in iters]
        for kind, key in ((0, "status_primal"), (1, "status_dual")):
            assert fg.fftgal_outcome(plan.handle, kind) == res[key]
        assert np.all(np.linalg.eigvalsh(res["upper"] - res["lower"]) > 0)
    finally:
        plan.close()
