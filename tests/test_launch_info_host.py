"""hhlb_launch_info reports what is launched: one launch per class, and the
windows of the kernel that the class runs."""
import ctypes

import pytest

H = pytest.importorskip("paper_1708_03249_amd")


def _info(channels, precision=0):
    h = ctypes.c_void_p()
    arr = (H._CChannel * len(channels))(*[c._c() for c in channels])
    assert H.lib().hhlb_create(arr, len(channels), precision, None, ctypes.byref(h)) == 0
    n, w = ctypes.c_int32(), ctypes.c_int64()
    assert H.lib().hhlb_launch_info(h, ctypes.byref(n), ctypes.byref(w)) == 0
    H.lib().hhlb_destroy(h)
    return n.value, w.value


@pytest.mark.parametrize("ch,windows", [
    # two cells per lane: 124 cells in one window, 234 in two, 110 more each
    (dict(Q=4, Nx=61), 1), (dict(Q=4, Nx=124), 1), (dict(Q=8, Nx=153), 2), (dict(Q=8, Nx=234), 2),
    (dict(Q=16, Nx=344), 3), (dict(Q=16, Nx=345), 4), (dict(quad=H.FULL_HERMITE, Q=8, Nx=454), 4),
    # one cell per lane where that takes a tenth fewer positions: 60, 106, 46 more each
    (dict(Q=4, Nx=60), 1), (dict(Q=8, Nx=125), 3), (dict(Q=12, Nx=152), 3), (dict(Q=16, Nx=244), 5),
    # f alone on the matrix cores: one cell per lane
    (dict(Q=16, transverse_dof=0, Nx=300), 7), (dict(Q=16, transverse_dof=0, Nx=107), 1),
    # the node-parallel stage: 58 cells
    (dict(Q=17, N=16, Nx=58), 1), (dict(Q=17, N=16, Nx=59), 2), (dict(quad=H.FULL_HERMITE, Q=40, N=20, Nx=117), 3),
])
def test_windows_of_one_channel(ch, windows):
    assert _info([H.Channel(**ch)]) == (1, windows)


def test_windows_add_up():
    chans = [H.Channel(Q=4, Nx=60), H.Channel(Q=8, Nx=234), H.Channel(Q=8, Nx=300), H.Channel(Q=17, N=16, Nx=59)]
    assert _info(chans) == (3, 1 + 2 + 3 + 2)
