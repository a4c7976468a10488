"""The sigma_0 stage in the FP64 FMA launches, at both sides of the rules that
say how it rides along: all workgroups on the GPU at once or not (1280 tiles),
its rows in LDS or read from memory, above 48 states with more modes than
states (a launch of its own).  Right-hand sides against the FP64 oracle, general
states.  Tolerance 1e-12 of the largest element."""

import numpy as np
import pytest

import heom_inputs as hi

pytestmark = pytest.mark.gpu

# (N, baths, Matsubara terms, depth, complex H)
SIZES = [
    (14, 14, 0, 3, False),  # 679 tiles: rows in LDS beyond 8 KiB
    (14, 13, 0, 4, False),  # 2379 tiles: from memory
    (20, 20, 0, 2, True),   # 230
    (20, 20, 0, 3, True),   # 1770
    (9, 9, 0, 5, True),     # 2001: rows within 8 KiB
    (52, 13, 3, 1, False),  # 52 modes: rides along
    (52, 27, 1, 1, False),  # 54: its own launch
    (49, 5, 0, 6, True),    # rides along without rows
]


@pytest.mark.parametrize("size", SIZES, ids=[str(s) for s in SIZES])
def test_right_hand_side_matches_oracle(orc, size):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_03498_amd as heom
    N, nb, M, D, hc = size
    print("CASE sigma_0", size, flush=True)
    prob = hi.random_problem(60 + N + D, N, n_baths=nb, M=M, D=D, complex_h=hc)
    h = heom.Hierarchy(prob, heom.FP64)
    x = hi.random_state(61 + N, h.n_ado, N, scale=0.1)
    want = orc.rhs(prob, x)
    a, b = h.state_from_numpy(x), h.new_state()
    h.rhs(a, b, hermitian=False)
    torch.cuda.synchronize()
    assert np.max(np.abs(h.state_to_numpy(b) - want)) <= 1e-12 * max(1.0, np.max(np.abs(want)))
