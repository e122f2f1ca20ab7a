"""The step kernel (whole RK-3 steps per launch, 128-cell windows) where its
window rules change, against the oracle: one window up to 124 cells, two from
125 to 234, 110 more each; walls at odd and even positions; channels of one
window, which take many steps in one launch, beside longer ones in one solver;
launches of up to 64 steps and their remainders.

Tolerance: 1e-12, the FP64 bar of the parity tests."""
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


def _check(chans, nsteps, tuning=None, what=""):
    states = initial_states(chans, seed=41, perturb=0.03)
    gpu = run_gpu(chans, states, nsteps, tuning=tuning)
    assert gpu["bad"] == 0
    compare(chans, gpu, run_oracle(chans, states, nsteps, gpu["dt"]), tol=1e-12, what=what)


@pytest.mark.parametrize("quad,Q,dof", [("HALF_HERMITE", 4, 2), ("HALF_HERMITE", 16, 2), ("HALF_HERMITE", 8, 0),
                                        ("FULL_HERMITE", 8, 2)])
def test_window_edges(quad, Q, dof):
    import paper_1708_03249_amd as H
    lengths = (8, 9, 123, 124, 125, 126, 127, 233, 234, 235, 344, 345, 454, 564, 565)
    chans = [H.Channel(quad=getattr(H, quad), Q=Q, Nx=nx, adv=H.WENO5, transverse_dof=dof, stretch_A=0.5 * (k % 2),
                       Kn=0.05 * (1 + k % 3), g=-0.4, T_right=1.3, dt=-0.5) for k, nx in enumerate(lengths)]
    _check(chans, 4, what=f"{quad} Q={Q}: windows of {lengths}")


@pytest.mark.parametrize("graph", [0, 70])
def test_many_steps_per_launch(graph):
    """131 steps of a class of one-window channels (launches of 64, 64 and 3
    steps; or a 70-step graph and single steps) beside a class of longer
    channels that takes one step per launch."""
    import paper_1708_03249_amd as H
    chans = [H.Channel(Q=4, Nx=nx, adv=H.UPWIND3, Kn=0.1, g=-0.2, T_right=1.2, dt=5e-4) for nx in (64, 117)]
    chans += [H.Channel(Q=3, Nx=nx, adv=H.WENO5, Kn=0.2, g=-0.3, dt=5e-4) for nx in (40, 150)]
    _check(chans, 131, tuning=dict(graph_steps=graph), what=f"131 steps, graphs of {graph}")


@pytest.mark.parametrize("adv", ["WENO5", "UPWIND3"])
def test_vanishing_differences(adv):
    """Uniform stretches next to perturbed cells: smoothness indicators that
    are zero, tiny or mixed send lanes through the rescaled weights and the
    limit rule."""
    import numpy as np
    import paper_1708_03249_amd as H
    chans = [H.Channel(Q=4, Nx=130, adv=getattr(H, adv), Kn=0.1, g=-0.2, T_right=1.2, dt=-0.5)]
    states = initial_states(chans, seed=3)
    for k, y in enumerate(states[0]):
        y[:, 20 + k] *= 1.0 + 1e-3
        y[:, 60:63] *= 1.0 + 1e-150
        y[:, 90] *= 1.0 + 1e-12
        y[:, 110:] = y[:, 110:] * np.float64(1.25)
    gpu = run_gpu(chans, states, 6)
    assert gpu["bad"] == 0
    compare(chans, gpu, run_oracle(chans, states, 6, gpu["dt"]), tol=1e-12, what=f"flat stretches, {adv}")


@pytest.mark.parametrize("form", ["mixed_f32", "mixed_bf16", "mixed_f16"])
@pytest.mark.parametrize("Q,dof,nsteps", [(4, 2, 4), (16, 2, 4), (12, 0, 4), (3, 2, 131)])
def test_mixed_window_edges(form, Q, dof, nsteps):
    """The mixed step kernel at the same edges (lengths of one, two and more
    windows; with nsteps = 131 one-window channels that keep their correction
    words in registers through launches of 64, 64 and 3 steps), one channel
    with a uniform stretch.  Tolerance: 1e-5 in n, u and T, the bar of the
    mixed forms (each stage rounds faces and increments to FP32, 6e-8)."""
    import paper_1708_03249_amd as H
    from gpu_common import moment_errors
    lengths = (8, 123, 124) if nsteps > 64 else (9, 124, 125, 127, 234, 235, 344, 345)
    chans = [H.Channel(Q=Q, Nx=nx, adv=H.WENO5, transverse_dof=dof, stretch_A=0.5 * (k % 2), Kn=0.05 * (1 + k % 3),
                       g=-0.4, T_right=1.3, dt=-0.5) for k, nx in enumerate(lengths)]
    states = initial_states(chans, seed=43, perturb=0.02)
    for y in states[1]:
        if y is not None:
            y[:, 30:60] = y[:, 30:31]
    gpu = run_gpu(chans, states, nsteps, precision=H.PRECISIONS[form])
    assert gpu["bad"] == 0
    e = moment_errors(chans, gpu, run_oracle(chans, states, nsteps, gpu["dt"]))
    assert max(e.values()) <= 1e-5, (form, e)


@pytest.mark.parametrize("quad,Q,dof,adv", [("HALF_HERMITE", 6, 0, "WENO5"), ("HALF_HERMITE", 8, 2, "WENO5"),
                                            ("HALF_HERMITE", 12, 2, "UPWIND3"), ("HALF_HERMITE", 16, 2, "WENO5"),
                                            ("HALF_HERMITE", 16, 0, "WENO5"), ("FULL_HERMITE", 16, 2, "WENO5")])
@pytest.mark.parametrize("over", [0, 1])
def test_few_and_many_windows(quad, Q, dof, adv, over):
    """The FP64 kernel's two forms on either side of the launch size where they
    change: as many one-window channels as the few-window form takes (512
    windows of four waves at two waves per SIMD, half of that at Q = 16, twice
    that for f alone), and one more.  The first, a middle and the last channel
    against the oracle."""
    import paper_1708_03249_amd as H
    n = 512 // (2 if quad == "HALF_HERMITE" and Q == 16 else 1) * (1 if dof else 2) + over
    chans = [H.Channel(quad=getattr(H, quad), Q=Q, Nx=16, adv=getattr(H, adv), transverse_dof=dof,
                       Kn=0.05 * (1 + k % 3), g=-0.4, T_right=1.3, dt=-0.5) for k in range(n)]
    states = initial_states(chans, seed=53, perturb=0.03)
    gpu = run_gpu(chans, states, 3)
    assert gpu["bad"] == 0
    ref = run_oracle(chans, states, 3, gpu["dt"], which=[0, n // 2, n - 1])
    compare(chans, gpu, ref, tol=1e-12, what=f"{quad} Q={Q} dof={dof}: {n} windows")
