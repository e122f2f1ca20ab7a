"""The temperature of full-range channels (at most 16 nodes) far from rest:
u = 3, T = 0.2 in units of the nodes' width, so that sum p^2 f is 46 times the
thermal part n T.  One RK-3 step of dt = Kn/2 with advection made negligible by
a long channel; what is left is the collision, which carries an error of T into
the populations (through about 0.9 of the largest one per relative change of T).

Tolerance: 20 eps of a cell's largest population, against the oracle.  With the
energy summed about u its rounding moves a population by at most 8 eps (256
random cells in 64-bit arithmetic against 80-bit) in the kernel and in the
oracle each, and 4 eps are left for the rest of the step; from raw sums,
sum p^2 f - u sum p f, it is 58 eps."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_common import initial_states, run_gpu, run_oracle  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("nx", [120, 300])
def test_energy_about_the_mean_velocity(nx):
    import paper_1708_03249_amd as H
    ch = H.Channel(quad=H.FULL_HERMITE, Q=16, N=15, Nx=nx, adv=H.UPWIND3, transverse_dof=0, L=1e6 * nx, Kn=0.1,
                   g=0.0, dt=0.05)
    (state,) = initial_states([ch], seed=61, perturb=0.02, u0=3.0, T0=0.2)
    gpu = run_gpu([ch], [state], 1)
    ref = run_oracle([ch], [state], 1, gpu["dt"])[0]
    f, r = gpu["f"].reshape(ch.V, nx), ref["f"]
    e = np.max(np.abs(f - r) / np.abs(r).max(axis=0))
    print(f"Nx={nx}: {e / 2.2e-16:.1f} eps", flush=True)
    assert e <= 20 * 2.2e-16, e
