"""Mixed forms with at most four nodes per half contract the force block in FP32
whatever the operand format asked for: the BF16 and FP16 forms give the FP32
form's bits.  From six nodes on their operands are their own."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_common import initial_states, run_gpu  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("Q,dof", [(1, 2), (2, 0), (3, 2), (4, 2), (4, 0), (6, 2)])
def test_small_blocks_in_fp32(Q, dof):
    import paper_1708_03249_amd as H
    chans = [H.Channel(Q=Q, Nx=nx, adv=H.WENO5, transverse_dof=dof, Kn=0.1, g=-0.4, T_right=1.3, dt=-0.5)
             for nx in (40, 117, 300)]
    states = initial_states(chans, seed=95, perturb=0.02)
    ref, *others = [run_gpu(chans, states, 5, precision=H.PRECISIONS[form])
                    for form in ("mixed_f32", "mixed_bf16", "mixed_f16")]
    for other in others:
        same = all(np.array_equal(ref[k], other[k]) for k in ("f", "chi", "n", "u", "T", "nw"))
        assert same == (Q <= 4), Q
