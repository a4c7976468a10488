"""The stage kernels by name, at sizes that runs otherwise take in one launch,
packed or in tiles: against the FP64 oracle, the step graph against direct
launches, and workspaces full of NaN and other launch shapes (the last two bit
for bit).  Every case asserts the kernel that it is about.

Tolerances: FP64 1e-12 of the largest element over 3 steps, FP32 1e-5 (the
rounding of FP32 storage, 6e-8, over 12 stages, and sums over up to W + D
neighbours)."""

import numpy as np
import pytest

import heom_inputs as hi
import run_forms as rf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def heom():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1803_03498_amd as heom
    heom.load()
    return heom


# (kernel, N, baths, Matsubara terms, depth, precision, Hermitian, complex H)
CASES = [
    ("k_bulk_fma", 7, 7, 1, 4, 1, True, False),
    ("k_bulk_fma", 7, 7, 1, 4, 0, True, False),
    ("k_bulk_fma", 8, 7, 1, 3, 0, False, False),
    ("k_bulk_fma", 9, 9, 1, 2, 1, True, True),
    ("k_bulk_fma", 14, 14, 0, 3, 0, True, False),
    ("k_bulk_fma", 18, 18, 0, 2, 0, True, True),
    ("k_stage_small", 8, 8, 1, 6, 1, True, False),
    ("k_stage_small", 8, 8, 1, 6, 0, True, False),
    ("k_stage_small", 12, 4, 1, 10, 0, True, False),
    ("k_stage_small", 16, 8, 0, 10, 0, True, True),  # N^2 = 256, the largest divisor of its index decode
    ("k_bulk_mfma", 16, 16, 0, 3, 0, True, False),
    ("k_bulk_mfma", 20, 20, 0, 2, 0, True, False),
    ("k_bulk_mfma", 33, 33, 0, 2, 0, True, False),
    ("k_stage_persist", 12, 12, 1, 2, 1, True, False),
    ("k_stage_persist", 16, 16, 0, 3, 1, True, False),
    ("k_stage_persist", 22, 22, 0, 2, 1, True, False),
    ("k_bulk_mfma_pk", 24, 24, 0, 3, 2, True, False),
]
IDS = [f"{c[0]}-{c[1:]}" for c in CASES]


def _problem(case):
    kernel, N, nb, M, D, precision, herm, hc = case
    prob = hi.random_problem(1000 + N + D, N, n_baths=nb, M=M, D=D, complex_h=hc)
    assert rf.run_kernel(prob, precision, herm) == kernel
    return prob


def _state(h, case):
    _, N, *_, precision, herm, _ = case
    x = hi.random_state(1100 + N, h.n_ado, N, hermitian=herm, scale=0.1)
    if precision:
        x[1:] = x[1:].astype(np.complex64)
    return x


@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_run_matches_oracle(heom, orc, case):
    print("CASE stage kernel", case, flush=True)
    N, precision, herm, dt, steps = case[1], case[5], case[6], 0.1, 3
    if (case[1], case[4]) == (16, 10):
        steps = 1
    with rf.stages_only():
        prob = _problem(case)
        h = heom.Hierarchy(prob, precision)
        x = _state(h, case)
        y, rec_ref = orc.propagate(prob, x, dt, steps, 1, {"kind": "population"})
        st = h.state_from_numpy(x)
        rec = h.propagate(st, dt, steps, 1, hermitian=herm)
    tol = 1e-12 if precision == 0 else 1e-5
    assert np.max(np.abs(h.state_to_numpy(st) - y)) <= tol * max(1.0, np.max(np.abs(y)))
    assert np.max(np.abs(rec[:, :N + 2] - rec_ref[:, :N + 2])) <= tol * max(1.0, np.max(np.abs(rec_ref)))


def _run(heom, h, x, case, steps, timing=False, fill=0):
    lib = heom.load()
    st = h.state_from_numpy(x)
    work = h.workspace(steps, 2, 0)
    work.fill_(fill)
    lib.heom_timing_enable(1 if timing else 0)
    try:
        rec = h.propagate(st, 0.1, steps, 2, hermitian=case[6], work=work)
    finally:
        lib.heom_timing_enable(0)
        lib.heom_timing_read(None, None, None, 1)
    return (rec,) + h.get_state(st)


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_graph_poison_and_launch_shape(heom, case):
    """Direct launches (timing on) against graph replays with the program's own
    work between them; a workspace of NaN; three workers, one ADO per tile."""
    import torch
    print("CASE stage kernel bits", case, flush=True)
    with rf.stages_only():
        h = heom.Hierarchy(_problem(case), case[5])
        x = _state(h, case)
        direct = _run(heom, h, x, case, 12, timing=True)
        assert np.all(np.isfinite(direct[0]))
        for fill in (0, 255):
            a = torch.randn(256, 256, device="cuda")
            (a @ a).sum().item()
            assert _same(direct, _run(heom, h, x, case, 12, fill=fill))
        heom.set_launch_shape(max_workgroups=3, max_ados_per_tile=1)
        try:
            assert _same(direct, _run(heom, h, x, case, 12, fill=255))
        finally:
            heom.set_launch_shape(0, 0)


# sizes of the packed form's edges whose workspace does hold the packed arrays (it
# does where the depth is at most the number of modes), smaller ones held off the
# resident form: one row block with whole and with broken rows, two groups of
# links at even and odd N
PACKED = [(13, 4, 1, 3, 0), (14, 14, 0, 2, 0), (15, 5, 0, 5, 0), (16, 5, 0, 4, 0), (18, 6, 0, 6, 0), (18, 6, 0, 6, 1),
          (29, 5, 0, 5, 0), (29, 5, 0, 5, 1), (29, 5, 0, 5, 2), (43, 5, 0, 5, 0), (43, 5, 0, 5, 1), (43, 5, 0, 5, 2),
          (48, 5, 0, 5, 0), (47, 5, 0, 5, 1), (64, 5, 0, 5, 1)]


@pytest.mark.parametrize("size", PACKED, ids=[str(s) for s in PACKED])
def test_packed_run_matches_oracle(heom, orc, size):
    N, nb, M, D, precision = size
    print("CASE packed", size, flush=True)
    dt, steps = 0.05, 2
    with rf.forms(resident=False, packed_min=0):
        prob = hi.random_problem(1200 + N, N, n_baths=nb, M=M, D=D)
        assert rf.run_kernel(prob, precision) == "k_packed"
        h = heom.Hierarchy(prob, precision)
        x = hi.random_state(1300 + N, h.n_ado, N, hermitian=True, scale=0.1)
        if precision:
            x[1:] = x[1:].astype(np.complex64)
        y, rec_ref = orc.propagate(prob, x, dt, steps, 1, {"kind": "population"})
        st = h.state_from_numpy(x)
        work = h.workspace(steps, 1, 0)
        work.fill_(255)
        rec = h.propagate(st, dt, steps, 1, hermitian=True, work=work)
    tol = 1e-12 if precision == 0 else 1e-5
    assert np.max(np.abs(h.state_to_numpy(st) - y)) <= tol * max(1.0, np.max(np.abs(y)))
    assert np.max(np.abs(rec[:, :N + 2] - rec_ref[:, :N + 2])) <= tol * max(1.0, np.max(np.abs(rec_ref)))
