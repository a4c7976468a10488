"""Large Hermitian hierarchies of 2 to 8 states (k_columns) against the FP64
oracle: every N, more links than states (several chunks of N links), one and
several modes per state, states without modes, tiles whose element count is
odd, a last tile that is not full.  The sizes lie just above what one resident
launch holds.

Tolerances: FP64 1e-12 of the largest element over 3 steps; FP32 storage 1e-5."""

import ctypes

import numpy as np
import pytest

import heom_inputs as hi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def heom():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_03498_amd as heom
    heom.load()
    return heom


@pytest.fixture
def columns(heom):
    lib = heom.load()
    lib.heom_test_columns_min.argtypes = [ctypes.c_int64]
    lib.heom_test_columns_min.restype = None
    lib.heom_test_columns_min(1)
    yield
    lib.heom_test_columns_min(-1)


# (N, baths, Matsubara terms, depth)
SIZES = [
    (2, 2, 3, 13),
    (3, 3, 2, 10),
    (4, 2, 5, 7),
    (5, 5, 1, 8),
    (6, 6, 1, 6),
    (7, 7, 0, 9),
    (8, 8, 0, 8),
]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("size", SIZES, ids=[str(s) for s in SIZES])
def test_columns_run_matches_oracle(heom, orc, columns, size, precision):
    N, nb, M, D = size
    print("CASE columns", size, precision, flush=True)
    steps, dt = 3, 0.1
    run = hi.random_problem(800 + N, N, n_baths=nb, M=M, D=D)
    h = heom.Hierarchy(run, precision)
    assert h.n_ado * N * N > 256 * 2048
    x = hi.random_state(900 + N, h.n_ado, N, hermitian=True, scale=0.1)
    if precision:
        x[1:] = x[1:].astype(np.complex64)
    y, rec_ref = orc.propagate(run, x, dt, steps, 1, {"kind": "population"})
    st = h.state_from_numpy(x)
    work = h.workspace(steps, 1, 0)
    work.fill_(255)  # NaN: nothing is read that was not written
    rec = h.propagate(st, dt, steps, 1, hermitian=True, work=work)
    tol = 1e-12 if precision == 0 else 1e-5
    got = h.state_to_numpy(st)
    assert np.max(np.abs(got - y)) <= tol * max(1.0, np.max(np.abs(y)))
    assert np.max(np.abs(rec[:, :N + 2] - rec_ref[:, :N + 2])) <= tol * max(1.0, np.max(np.abs(rec_ref)))


@pytest.mark.parametrize("precision", [0, 1])
def test_columns_run_does_not_depend_on_the_launch_shape(heom, columns, precision):
    """Three workgroups instead of a full GPU, and a run (a step graph, but for
    its first and last step) split in two calls without one."""
    print("CASE columns shape", precision, flush=True)
    run = hi.random_problem(88, 7, M=0, D=9)
    h = heom.Hierarchy(run, precision)
    x = hi.random_state(89, h.n_ado, 7, hermitian=True, scale=0.1)
    out = []
    for cap, parts in ((0, [12]), (3, [12]), (0, [5, 7])):
        st = h.state_from_numpy(x)
        heom.set_launch_shape(max_workgroups=cap)
        try:
            for n in parts:
                rec = h.propagate(st, 0.1, n, n, hermitian=True)
        finally:
            heom.set_launch_shape()
        out.append((rec[-1], h.state_to_numpy(st)))
    for r, s in out[1:]:
        assert np.array_equal(r, out[0][0]) and np.array_equal(s, out[0][1])
