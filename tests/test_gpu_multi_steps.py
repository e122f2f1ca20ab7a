"""The whole-step kernel of the homogeneous mixed-quadrature system (App. A)
over its lane layouts, against the numpy oracle: every V_x with an instance;
2 to 64 lanes per point, powers of two and others (waves with spare lanes),
z axes of four velocities (lane permutations) and others, equilibrium orders in
each range (up to 3, 7, 20); and sets without an instance, which run the
per-stage kernel.  Launches of up to 64 steps give the bits of single steps.

Tolerance: 1e-12 of a point's scale, the bar of the other App. A tests."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from oracle import multi as M  # noqa: E402
from test_gpu_multi import TOL, _axes, _state  # noqa: E402

pytestmark = pytest.mark.gpu

HALF, FULL, LAG = 0, 1, 2


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


SETS = [  # (name, axes)
    ("V_x 4, 2 lanes", [(HALF, 2, 1, 1.0), (FULL, 2, 1, 1.0)]),
    ("V_x 4, 64 lanes", [(FULL, 4, 3, 1.0), (HALF, 4, 3, 1.0), (HALF, 4, 2, 1.0)]),
    ("V_x 6, 6 lanes", [(HALF, 3, 2, 1.0), (HALF, 3, 2, 1.0)]),
    ("V_x 8, 16 lanes", [(HALF, 4, 3, 1.0), (FULL, 4, 3, 1.0), (FULL, 4, 3, 1.0)]),
    ("V_x 8, 32 lanes, order 7", [(FULL, 8, 7, 1.0), (FULL, 4, 3, 1.0), (HALF, 4, 3, 1.0)]),
    ("V_x 10, 24 lanes", [(HALF, 5, 4, 1.0), (FULL, 6, 5, 1.0), (HALF, 2, 1, 1.0)]),
    ("V_x 12, 16 lanes, order 11", [(FULL, 12, 11, 1.0), (HALF, 8, 7, 1.0)]),
    ("V_x 16, 8 lanes", [(HALF, 8, 7, 1.0), (FULL, 8, 7, 1.0)]),
    ("V_x 20, 4 lanes, order 9", [(HALF, 10, 9, 1.0), (FULL, 4, 3, 1.0)]),
    ("V_x 24, 12 lanes", [(HALF, 12, 11, 1.0), (LAG, 3, 2, 0.6), (FULL, 2, 1, 1.0)]),
    ("V_x 2 (per stage)", [(FULL, 2, 1, 1.0), (HALF, 4, 3, 1.0), (FULL, 4, 3, 1.0)]),
    ("V_x 32 (per stage)", [(HALF, 16, 15, 1.0), (FULL, 4, 3, 1.0)]),
    ("128 lanes (per stage)", [(FULL, 4, 3, 1.0), (HALF, 4, 3, 1.0), (HALF, 8, 7, 1.0)]),
]


@pytest.mark.parametrize("name,spec", SETS, ids=[s[0] for s in SETS])
def test_every_lane_layout(name, spec):
    import torch
    import paper_1708_03249_amd as H
    haxes, oaxes = _axes(spec)
    F, npts, Kn, dt = np.array([0.4, -0.6, 0.3])[:len(spec)], 149, 0.3, 2e-3
    f = _state(oaxes, npts, 31)
    s = H.MultiSolver(haxes, npts, F, Kn)
    fd = torch.from_numpy(f).cuda()
    Ld = torch.empty_like(fd)
    s.rhs(fd, Ld)
    s.step(fd, dt, 3)
    torch.cuda.synchronize()
    ref = M.rhs(oaxes, f, F, Kn)
    scale = np.abs(ref).max(axis=1) + np.abs(f).max(axis=1) * f.sum(axis=1) / Kn
    assert np.max(np.abs(Ld.cpu().numpy() - ref) / scale[:, None]) < TOL
    ref = M.run(oaxes, f, F, Kn, dt, 3)
    assert np.max(np.abs(fd.cpu().numpy() - ref) / np.abs(ref).max(axis=1, keepdims=True)) < TOL


def test_launches_of_many_steps():
    """131 steps in one call (launches of 64, 64 and 3) and as single steps,
    bit for bit, also through the entry point without a workspace."""
    import torch
    import paper_1708_03249_amd as H
    spec = [(HALF, 4, 3, 1.0), (FULL, 4, 3, 1.0), (FULL, 4, 3, 1.0)]
    haxes, oaxes = _axes(spec)
    F, npts, Kn, dt = np.array([0.3, -0.2, 0.5]), 61, 0.2, 1e-3
    f0 = torch.from_numpy(_state(oaxes, npts, 33)).cuda()
    s = H.MultiSolver(haxes, npts, F, Kn)
    a, b, c = f0.clone(), f0.clone(), f0.clone()
    s.step(a, dt, 131)
    for _ in range(131):
        s.step(b, dt, 1)
    H.multi_step_noalloc(haxes, c, F, Kn, dt, 131)
    torch.cuda.synchronize()
    assert torch.isfinite(a).all() and torch.equal(a, b) and torch.equal(a, c)
