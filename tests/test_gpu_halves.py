"""GPU: the inverse x/y pass in two halves, on as many planes as it is taken for:
equal to the split passes byte for byte, and to the FP64 oracle within the bar
of the parity tests."""
import numpy as np
import pytest

from psatd_cases import random_fields, say
from test_gpu_parity import check, run_both
from test_gpu_rings import rerun, state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,g", [((210, 201, 36), (3, 12, 2)), ((420, 1, 40), (0, 87, 1)), ((256, 192, 30), (0, 0, 0))])
def test_inverse_pass_in_halves(N, g):
    """Padded planes of 216 x 225 (odd interior rows), 420 x 175 with one interior
    row, and 256 x 192 (two stages each way); the fused exchange keeps the split
    passes."""
    import torch
    say(f"inverse pass in halves, {N} guards {g}")
    E, B, J = (x.astype(np.float32).astype(np.float64) for x in random_fields(N, 52, p=8))
    case, eE, eB, _ = run_both(N, [[0, 0, 0]], [list(N)], [g], 8, 0.5, 1.0, "f32", "replicated", (E, B, J), 2)
    assert case.plan.tuning()["split_xy"] == 1
    check(case, eE, eB, "f32", 1e-5)
    first = state(case)
    assert torch.equal(first, rerun(case, E, B, lambda c: None, 2, fuse_eb=1))
