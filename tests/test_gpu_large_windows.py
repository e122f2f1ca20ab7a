"""The node-parallel stage (Q > 16) where its windows change, against the
oracle: 26 cells and fewer fill two 16-cell blocks of the contraction, 27 and
more take four, 59 split into two windows, 117 into three; partial sums
carried from stage to stage over several calls of several steps; tiles whose
last wave has one node or none; channels of both kinds (colliding or not) in
one class.

Tolerance: 1e-12, the FP64 bar of the parity tests."""
import math
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_common import compare, initial_states, run_gpu, run_oracle  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("quad,Q,dof,adv", [("HALF_HERMITE", 17, 2, "WENO5"), ("HALF_HERMITE", 31, 0, "UPWIND3"),
                                            ("FULL_HERMITE", 38, 2, "WENO5"), ("FULL_HERMITE", 18, 0, "WENO5")])
@pytest.mark.parametrize("graph,lengths", [(0, (8, 25, 26)), (3, (27, 58, 59, 60, 116, 117))])
def test_large_windows(quad, Q, dof, adv, graph, lengths):
    import paper_1708_03249_amd as H
    chans = [H.Channel(quad=getattr(H, quad), Q=Q, N=min(20, Q - 1), Nx=nx, adv=getattr(H, adv), transverse_dof=dof,
                       stretch_A=0.5 * (k % 2), Kn=math.inf if k % 3 == 1 else 0.1 * (1 + k % 2), g=-0.1,
                       T_right=1.2, dt=1e-4) for k, nx in enumerate(lengths)]
    states = initial_states(chans, seed=47, perturb=0.0)
    gpu = run_gpu(chans, states, 7, tuning=dict(graph_steps=graph))
    assert gpu["bad"] == 0
    compare(chans, gpu, run_oracle(chans, states, 7, gpu["dt"]), tol=1e-12, what=f"{quad} Q={Q} {lengths}")
