"""FP32 Hermitian runs on the persistent matrix-core kernel (hierarchies too
small for the packed form and too large for one launch) against the FP64
oracle, for one to four row blocks, element pairs (even N) and single elements
(odd N): with three bases in stage 4 (few ADOs of more than 16 states), and
with the one that stage 2 leaves.

Tolerance: 1e-5 of the largest element over 3 steps (FP32 storage)."""

import ctypes

import numpy as np
import pytest

import heom_inputs as hi

pytestmark = pytest.mark.gpu

# (N, baths, Matsubara terms, depth)
SIZES = [(15, 15, 0, 4), (16, 16, 0, 4), (24, 5, 0, 3), (31, 4, 0, 3), (35, 2, 1, 3), (48, 4, 0, 2), (63, 3, 0, 2),
         (64, 3, 0, 2), (18, 8, 1, 4), (35, 28, 0, 3), (50, 28, 0, 3), (51, 28, 0, 3)]


@pytest.mark.parametrize("size", SIZES, ids=[str(s) for s in SIZES])
def test_persistent_run_matches_oracle(orc, size):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_03498_amd as heom
    lib = heom.load()
    lib.heom_test_packed_min.argtypes = [ctypes.c_int64]
    lib.heom_test_packed_min.restype = None
    N, nb, M, D = size
    print("CASE persistent", size, flush=True)
    steps, dt = 3, 0.1
    run = hi.random_problem(300 + N, N, n_baths=nb, M=M, D=D)
    h = heom.Hierarchy(run, 1)
    x = hi.random_state(400 + N, h.n_ado, N, hermitian=True, scale=0.1)
    x[1:] = x[1:].astype(np.complex64)
    y, rec_ref = orc.propagate(run, x, dt, steps, 1, {"kind": "population"})
    st = h.state_from_numpy(x)
    work = h.workspace(steps, 1, 0)
    work.fill_(255)  # NaN: nothing is read that was not written
    lib.heom_test_packed_min(1 << 62)
    try:
        rec = h.propagate(st, dt, steps, 1, hermitian=True, work=work)
    finally:
        lib.heom_test_packed_min(-1)
    got = h.state_to_numpy(st)
    assert np.max(np.abs(got - y)) <= 1e-5 * max(1.0, np.max(np.abs(y)))
    assert np.max(np.abs(rec[:, :N + 2] - rec_ref[:, :N + 2])) <= 1e-5 * max(1.0, np.max(np.abs(rec_ref)))
