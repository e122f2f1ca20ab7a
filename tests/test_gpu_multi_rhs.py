"""The right-hand side of the homogeneous system (App. A) alone, on both sides of
the size where it changes kernels: with an axis order above 7, up to 64 blocks of
the whole-step kernel (of 64 // lanes-per-point points in each of four waves) run
the stage kernel.  Against the numpy oracle at the first and last points.

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


@pytest.mark.parametrize("spec,per_wave", [([(HALF, 10, 9, 1.0), (FULL, 4, 3, 1.0)], 16),
                                           ([(HALF, 12, 11, 1.0), (LAG, 3, 2, 0.6), (FULL, 2, 1, 1.0)], 5)])
@pytest.mark.parametrize("over", [0, 1])
def test_both_sides_of_the_rule(spec, per_wave, over):
    import torch
    import paper_1708_03249_amd as H
    haxes, oaxes = _axes(spec)
    F, Kn, npts = np.array([0.4, -0.6, 0.3])[:len(spec)], 0.3, 64 * 4 * per_wave + over
    f = _state(oaxes, npts, 35)
    s = H.MultiSolver(haxes, npts, F, Kn)
    Ld = torch.empty(f.shape, dtype=torch.float64, device="cuda")
    s.rhs(torch.from_numpy(f).cuda(), Ld)
    torch.cuda.synchronize()
    for part in (slice(0, 30), slice(npts - 30, npts)):
        ref = M.rhs(oaxes, f[part], F, Kn)
        scale = np.abs(ref).max(axis=1) + np.abs(f[part]).max(axis=1) * f[part].sum(axis=1) / Kn
        assert np.max(np.abs(Ld[part].cpu().numpy() - ref) / scale[:, None]) < TOL
