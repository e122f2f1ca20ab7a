"""The residual of a nearly steady state, max ||L[y]||_inf / ||y||_inf over f and
chi, against the oracle's right-hand side on the same state: the equilibrium at
rest, modulated by 1e-9 of itself along the channel, at dt = 1e-7.  Formed as
(y1 - y)/dt from a rounded y1 = y + dt L[y] it would be known to eps/dt of y
only, about a tenth of it.

Tolerance: 1e-4.  L is the difference of fluxes v y/dx; a few roundings of them
(eps times 5 times 120 cells times y) are 1e-13 y in a residual of about 1e-8
y, 1e-5 of it."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import oracle as O  # noqa: E402
from gpu_common import initial_states, to_oracle  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("quad,Q", [("HALF_HERMITE", 4), ("HALF_HERMITE", 16), ("FULL_HERMITE", 16),
                                    ("HALF_HERMITE", 17)])
def test_residual_near_the_steady_state(quad, Q):
    import torch
    import paper_1708_03249_amd as H
    chans = [H.Channel(quad=getattr(H, quad), Q=Q, N=min(20, Q - 1), Nx=nx, adv=H.UPWIND3, Kn=kn, g=0.0, dt=1e-7)
             for nx, kn in ((120, 0.1), (64, 1.0))]
    states = initial_states(chans)
    for (f, chi), ch in zip(states, chans):
        for y in (f, chi):
            y *= 1.0 + 1e-9 * np.sin(2 * np.pi * (np.arange(ch.Nx) + 0.5) / ch.Nx + np.arange(ch.V)[:, None])
    s = H.Solver(chans)
    s.set_state(*(torch.from_numpy(np.concatenate([st[k].ravel() for st in states])).cuda() for k in (0, 1)))
    res = s.diagnostics(residual=True)[3].cpu().numpy()
    f, chi = (x.cpu().numpy() for x in s.get_state())
    s.close()
    assert np.array_equal(f, np.concatenate([st[0].ravel() for st in states]))   # the state itself is as it was
    for k, (ch, (fk, ck)) in enumerate(zip(chans, states)):
        Lf, Lc, _ = O.rhs(to_oracle(ch), fk, ck)
        r = max(np.abs(Lf).max() / np.abs(fk).max(), np.abs(Lc).max() / np.abs(ck).max())
        print(f"{quad} Q={Q} Nx={ch.Nx}: residual {res[k]:.6e}, oracle {r:.6e}", flush=True)
        assert abs(res[k] / r - 1) < 1e-4, (k, res[k], r)
