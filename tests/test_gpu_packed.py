"""Hermitian propagation in packed form (k_packed) against the FP64 oracle, at
the edges of its tiles: N = 16 k + 1, 4 k, 16 k, odd N, the last K block of 1
to 16 columns, one and several groups of four "-" links, several modes per
state, no level below the top (depth 1), fewer ADOs than wavefronts, side rows
and (where the workspace has no room for them) none.

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
def packed(heom):
    lib = heom.load()
    lib.heom_test_packed_min.argtypes = [ctypes.c_int64]
    lib.heom_test_packed_min.restype = None
    lib.heom_test_packed_min(0)
    yield
    lib.heom_test_packed_min(-1)


# (N, baths, Matsubara terms, depth)
SIZES = [
    (10, 9, 0, 9),   # one row block, FP64 only; three groups of links
    (13, 4, 1, 3),
    (14, 14, 0, 2),
    (15, 5, 0, 5),
    (16, 3, 0, 4),
    (18, 6, 0, 6),   # two groups of links
    (23, 4, 0, 1),   # top level only; N odd, two row blocks
    (24, 24, 0, 2),  # 8 columns in the last block
    (25, 3, 2, 3),   # three modes per state
    (29, 2, 0, 7),   # deep, few ADOs
    (31, 31, 0, 2),
    (32, 32, 0, 2),  # whole tiles
    (33, 33, 0, 2),  # one column in the last block
    (36, 5, 1, 3),
    (43, 3, 0, 9),
    (47, 10, 0, 2),
    (48, 12, 1, 2),
    (49, 6, 0, 3),   # four row blocks (FP64 stays with the complex kernels)
    (60, 8, 0, 2),
    (64, 4, 0, 3),
]


CASES = [(s, p) for s in SIZES for p in (0, 1, 2) if p == 0 or s[0] >= 17]


@pytest.mark.parametrize("size, precision", CASES, ids=[f"{s}-{p}" for s, p in CASES])
def test_packed_run_matches_oracle(heom, orc, packed, size, precision):
    N, nb, M, D = size
    print("CASE packed", size, precision, flush=True)
    steps, dt = 3, 0.1
    run = hi.random_problem(500 + N, N, n_baths=nb, M=M, D=D)
    h = heom.Hierarchy(run, precision)
    x = hi.random_state(600 + N, h.n_ado, N, hermitian=True, scale=0.1)
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


@pytest.mark.parametrize("precision", [0, 1, 2])
def test_packed_run_does_not_depend_on_the_launch_shape(heom, packed, precision):
    """Three workgroups instead of one per CU, and runs split in two calls."""
    print("CASE packed shape", precision, flush=True)
    run = hi.random_problem(77, 33, M=0, D=3)
    h = heom.Hierarchy(run, precision)
    x = hi.random_state(78, h.n_ado, 33, hermitian=True, scale=0.1)
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
