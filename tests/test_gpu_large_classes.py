"""Classes of large velocity sets (Q > 16) beside each other and beside small
ones in one solver: every channel gives the bits it gives in a solver of its
own, in every launch configuration, read-outs and residual included.  A class
keeps its partial sums at an offset of its own, tiles and cells differ."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_common import initial_states  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _run(chans, states, tuning):
    import torch
    import paper_1708_03249_amd as H
    s = H.Solver(chans)
    s.set_tuning(**tuning)
    s.set_state(*(torch.from_numpy(np.concatenate([st[k].ravel() for st in states])).cuda() for k in (0, 1)))
    s.step(3)
    s.step(2)
    f, chi = (x.cpu().numpy() for x in s.get_state())
    mom = [x.cpu().numpy() for x in s.moments()]
    nw, mass, bad, res = (x.cpu().numpy() for x in s.diagnostics(residual=True))
    assert int(bad.sum()) == 0
    out = []
    for c in range(len(chans)):
        o, a = slice(s.offsets[c], s.offsets[c + 1]), slice(s.cells[c], s.cells[c + 1])
        out.append([f[o], chi[o], *(m[a] for m in mom), nw[c], mass[c], res[c]])
    s.close()
    return out


@pytest.mark.parametrize("tuning", [dict(), dict(class_streams=1), dict(graph_steps=2), dict(merge_classes=1)],
                         ids=["direct", "streams", "graph", "merged"])
def test_classes_together_and_apart(tuning):
    import paper_1708_03249_amd as H
    kw = dict(adv=H.WENO5, g=-0.1, T_right=1.2, dt=1e-4)
    chans = [H.Channel(Q=4, Nx=300, Kn=0.1, **kw), H.Channel(Q=40, N=20, Nx=70, Kn=0.2, **kw),
             H.Channel(quad=H.FULL_HERMITE, Q=18, Nx=33, Kn=0.1, **kw), H.Channel(Q=12, Nx=100, Kn=0.3, **kw),
             H.Channel(Q=17, Nx=130, Kn=0.1, **kw), H.Channel(Q=40, N=20, Nx=24, Kn=0.1, **kw)]
    states = initial_states(chans, seed=71)
    together = _run(chans, states, tuning)
    for c, ch in enumerate(chans):
        (apart,) = _run([ch], [states[c]], {})
        for x, y in zip(together[c], apart):
            assert np.array_equal(x, y), (c, np.abs(x - y).max())
