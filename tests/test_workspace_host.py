"""Workspace of solvers that mix velocity sets: channels of different model
classes in one solver need what each needs in a solver of its own, so a small
channel of a large set (whose stages keep partial sums per tile of 16 nodes and
cell) beside long channels of a small one costs what it costs alone."""
import ctypes

import pytest

H = pytest.importorskip("paper_1708_03249_amd")


def _bytes(channels, precision=0):
    h = ctypes.c_void_p()
    arr = (H._CChannel * len(channels))(*[c._c() for c in channels])
    assert H.lib().hhlb_create(arr, len(channels), precision, None, ctypes.byref(h)) == 0
    nb = ctypes.c_size_t()
    assert H.lib().hhlb_workspace_bytes(h, ctypes.byref(nb)) == 0
    H.lib().hhlb_destroy(h)
    return nb.value


@pytest.mark.parametrize("large", [dict(Q=200), dict(Q=17), dict(quad=H.FULL_HERMITE, Q=500)])
@pytest.mark.parametrize("others", [[dict(Q=4, Nx=100000)], [dict(Q=18, Nx=20000), dict(Q=8, Nx=1000)]])
def test_classes_share_a_solver_at_no_cost(large, others):
    # f only in every channel: a solver with chi in one stores it for all
    small = [H.Channel(transverse_dof=0, **c) for c in others]
    big = [H.Channel(Nx=24, N=16, transverse_dof=0, **large)]
    apart, together = sum(_bytes([c]) for c in small + big), _bytes(small + big)
    assert together <= apart + 65536, (together, apart)
