"""The step kernels' windows of 64 cells, one per lane (short channels, and those
that two-cell windows fit badly), against the oracle: channels of one window up
to 60 cells, through launches of many steps; of three (125 to 152 cells) and
five (235 to 244); f alone at Q = 16, which takes them at every length up to
eight windows.  Walls in the first and last window, halos of nine cells inside.

Tolerance: 1e-12, the FP64 bar of the parity tests; for the mixed forms 1e-5 in
n, u and T (each stage rounds faces and increments to FP32, 6e-8)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_common import compare, initial_states, moment_errors, run_gpu, run_oracle  # noqa: E402

pytestmark = pytest.mark.gpu

ONE, SEVERAL, ANY = (8, 9, 37, 59, 60), (125, 126, 150, 152, 240, 244), (61, 106, 107, 153, 300)


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _channels(quad, Q, dof, adv, lengths):
    import paper_1708_03249_amd as H
    p0 = 0.3 if quad == "HALF_LAGUERRE" else 1.0
    return [H.Channel(quad=getattr(H, quad), Q=Q, N=min(4, Q - 1) if p0 < 1.0 else -1, Nx=nx, adv=getattr(H, adv),
                      transverse_dof=dof, stretch_A=0.5 * (k % 2), Kn=0.05 * (1 + k % 3), g=-0.4, T_right=1.3, p0=p0,
                      dt=-0.5) for k, nx in enumerate(lengths)]


@pytest.mark.parametrize("quad,Q,dof,adv", [
    ("HALF_HERMITE", 1, 2, "WENO5"), ("HALF_HERMITE", 4, 2, "UPWIND3"), ("HALF_HERMITE", 8, 0, "WENO5"),
    ("HALF_HERMITE", 12, 2, "WENO5"), ("HALF_HERMITE", 16, 2, "WENO5"), ("HALF_HERMITE", 16, 0, "WENO5"),
    ("FULL_HERMITE", 4, 0, "UPWIND3"), ("FULL_HERMITE", 16, 2, "WENO5"), ("HALF_LAGUERRE", 8, 2, "WENO5")])
@pytest.mark.parametrize("lengths,nsteps", [(ONE, 4), (ONE, 70), (SEVERAL, 4)])
def test_fp64(quad, Q, dof, adv, lengths, nsteps):
    chans = _channels(quad, Q, dof, adv, lengths)
    states = initial_states(chans, seed=83, perturb=0.03)
    gpu = run_gpu(chans, states, nsteps)
    assert gpu["bad"] == 0
    compare(chans, gpu, run_oracle(chans, states, nsteps, gpu["dt"]), tol=1e-12, what=f"{quad} Q={Q} {lengths}")


@pytest.mark.parametrize("adv", ["WENO5", "UPWIND3"])
def test_f_alone_at_every_length(adv):
    chans = _channels("HALF_HERMITE", 16, 0, adv, ANY)
    states = initial_states(chans, seed=85, perturb=0.03)
    gpu = run_gpu(chans, states, 5)
    assert gpu["bad"] == 0
    compare(chans, gpu, run_oracle(chans, states, 5, gpu["dt"]), tol=1e-12, what=f"Q=16, f, {ANY}")


@pytest.mark.parametrize("nch", [300, 1500])
def test_many_short_channels(nch):
    """Batches beyond the few-window form; the first, a middle and the last."""
    import paper_1708_03249_amd as H
    chans = [H.Channel(Q=(4, 8, 16)[k % 3], Nx=24 + k % 30, adv=H.WENO5, Kn=0.05 * (1 + k % 3), g=-0.4, T_right=1.3,
                       dt=-0.5) for k in range(nch)]
    states = initial_states(chans, seed=87, perturb=0.03)
    gpu = run_gpu(chans, states, 3)
    assert gpu["bad"] == 0
    which = [0, 1, 2, nch // 2, nch // 2 + 1, nch - 1]
    compare(chans, gpu, run_oracle(chans, states, 3, gpu["dt"], which=which), tol=1e-12, what=f"{nch} short channels")


@pytest.mark.parametrize("nx,Q,dof,n", [(16, 16, 2, 512), (16, 16, 0, 512), (64, 8, 2, 512), (64, 16, 2, 256)])
@pytest.mark.parametrize("over", [0, 1])
def test_few_and_many_windows(nx, Q, dof, n, over):
    """Both sides of the launch size where the few-window form ends, with one
    cell per lane (16 cells) and two (64 cells)."""
    import paper_1708_03249_amd as H
    chans = [H.Channel(Q=Q, Nx=nx, adv=H.WENO5, transverse_dof=dof, Kn=0.05 * (1 + k % 3), g=-0.4, T_right=1.3, dt=-0.5)
             for k in range(n + over)]
    states = initial_states(chans, seed=91, perturb=0.03)
    gpu = run_gpu(chans, states, 3)
    assert gpu["bad"] == 0
    ref = run_oracle(chans, states, 3, gpu["dt"], which=[0, n // 2, n + over - 1])
    compare(chans, gpu, ref, tol=1e-12, what=f"Q={Q} Nx={nx}: {n + over} windows")


@pytest.mark.parametrize("form", ["mixed_f32", "mixed_bf16", "mixed_f16"])
@pytest.mark.parametrize("Q,dof", [(2, 2), (4, 0), (12, 2), (16, 2), (16, 0)])
@pytest.mark.parametrize("lengths,nsteps", [(ONE, 70), (SEVERAL, 4)])
def test_mixed(form, Q, dof, lengths, nsteps):
    import paper_1708_03249_amd as H
    chans = _channels("HALF_HERMITE", Q, dof, "WENO5", lengths)
    states = initial_states(chans, seed=89, perturb=0.02)
    gpu = run_gpu(chans, states, nsteps, precision=H.PRECISIONS[form])
    assert gpu["bad"] == 0
    e = moment_errors(chans, gpu, run_oracle(chans, states, nsteps, gpu["dt"]))
    assert max(e.values()) <= 1e-5, (form, e)
