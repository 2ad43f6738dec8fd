"""CPU checks of the workspace sizes of plans that run their solves one at a time.

A server admits requests by the bytes of their plans.  A plan that holds one
buffer set solves there as a member of the batch, one solve after another, so
it must not ask for the room in which the solves of one call run at once.
"""

import os

import pytest


@pytest.fixture(scope="module")
def fg():
    from paper_1412_2033_amd import fftgal
    if not os.path.exists(fftgal.LIB_PATH):
        pytest.fail("libfftgal.so not built: run __graft_entry__.build()")
    fftgal.load_library()
    return fftgal


# (d, N, bytes of the layout of one solve: FP64, FP32 iterations)
LAYOUTS = (
    (2, (41, 41), 2392576, 2500608),
    (2, (365, 365), 30922752, 39449600),
    (3, (63, 63, 63), 181511680, 217458176),
)


def test_server_plans_of_one_buffer_set(fg):
    from paper_1412_2033_amd import serve
    srv = object.__new__(serve.Server)  # no device
    srv.concurrent = False
    for fast in (False, True):
        srv.fast_grid = fast
        for d, N, fp64, fp32 in LAYOUTS:
            for precision, n in (("fp64", fp64), ("fp32", fp32)):
                srv.precision = precision
                assert fg.fftgal_workspace_bytes(d, N, srv.flags_for(d, N)) <= n, (N, precision)


def test_one_at_a_time_is_the_layout_alone(fg):
    one = fg.ONE_AT_A_TIME
    for d, N, fp64, fp32 in LAYOUTS:
        for precision, n in ((fg.FP64, fp64), (fg.FP32_ITER, fp32)):
            least = fg.fftgal_workspace_bytes(d, N, precision | one)
            assert least <= n and least <= fg.fftgal_workspace_bytes(d, N, precision)
    for scheme in ("ga", "gani", "reduced"):
        assert 0 < fg.fftgal_workspace_bytes(2, (9, 9), one, scheme=scheme) <= \
            fg.fftgal_workspace_bytes(2, (9, 9), 0, scheme=scheme)
    assert fg.fftgal_workspace_bytes(2, (9, 9), one | fg.CONCURRENT) == 0
