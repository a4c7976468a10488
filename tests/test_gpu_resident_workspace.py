"""Resident runs in workspaces of exactly the planned size, with a guard behind
them: hierarchies whose stage copies have just room for the flags of their
workgroups, or not (those run stage by stage), against the FP64 oracle, every
record.  The host walks all sizes in test_resident_layout.py.

Tolerances: FP64 1e-12 of the largest element over at most 6 steps; FP32
storage 1e-5, its rounding 6e-8 accumulated over 4 x 6 stages."""

import numpy as np
import pytest

import heom_inputs as hi

pytestmark = pytest.mark.gpu

GUARD = 1 << 16

# (N, baths, Matsubara terms, depth, precision, dt)
SIZES = [
    (12, 12, 0, 1, 1, 0.1),  # 12 ADOs on 12 workgroups
    (20, 3, 0, 1, 1, 0.1),   # 3
    (3, 3, 2, 3, 1, 0.1),    # 219, 18 elements each
    (2, 2, 1, 8, 1, 0.05),   # 494 of 2 x 2: no room, stage by stage
    (2, 2, 3, 4, 1, 0.02),   # the same
    (2, 2, 0, 16, 0, 0.02),  # 152, deep
    (2, 2, 0, 19, 1, 0.02),
    (1, 1, 60, 2, 1, 0.002), # 1952 of 1 x 1
]


@pytest.mark.parametrize("size", SIZES, ids=[str(s) for s in SIZES])
def test_exact_workspace(orc, size):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_03498_amd as heom
    N, nb, M, D, precision, dt = size
    run = hi.random_problem(40 + N, N, n_baths=nb, M=M, D=D)
    h = heom.Hierarchy(run, precision)
    x = hi.random_state(50 + N, h.n_ado, N, hermitian=True, scale=0.1)
    if precision:
        x[1:] = x[1:].astype(np.complex64)
    tol = 1e-12 if precision == 0 else 1e-5
    for steps in (6, 1):
        print("CASE exact workspace", size, steps, flush=True)
        y, rec_ref = orc.propagate(run, x, dt, steps, 1, {"kind": "population"})
        need = h.work_bytes(steps, 1, 0)
        buf = torch.full((need + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
        for form in ("workspace", "noalloc"):
            st = h.state_from_numpy(x)
            if form == "workspace":
                rec = h.propagate(st, dt, steps, 1, hermitian=True, work=buf[:need])
            else:
                rec = h.propagate_noalloc(st, dt, steps, 1, hermitian=True)
            assert bool((buf[need:] == 0xA5).all()), form
            assert np.max(np.abs(h.state_to_numpy(st) - y)) <= tol * max(1.0, np.max(np.abs(y))), form
            assert np.max(np.abs(rec[:, :N + 2] - rec_ref[:, :N + 2])) <= tol * max(1.0, np.max(np.abs(rec_ref))), form
