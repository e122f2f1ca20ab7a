"""The autotuner's choice leaves the two switches that select nothing at their
defaults, so that a merged launch can still be set after it."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_switches_that_select_nothing():
    import paper_1708_03249_amd as H
    s = H.Solver([H.Channel(Q=Q, Nx=70, Kn=0.1, dt=1e-4) for Q in (4, 8)])
    s.init_equilibrium(1.0, 0.0, 1.0)
    for _ in range(8):   # by chance alone one of eight would differ
        best = s.autotune(trial_steps=1)
        assert (best["step_fusion"], best["waves_per_window"]) == (0, 2), best
    s.set_tuning(merge_classes=1)
    s.close()
