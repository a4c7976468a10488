"""Small hierarchies: a whole run in one launch (k_resident), against the FP64
oracle.  Sizes at the edges of its forms: one workgroup (one and two elements
per thread), a grid (one, two and four), N = 1 and N = 22, more coupling
entries per element than modes of two states usually give, general states,
complex H, a run longer than one launch takes, a launch that gives up its
waits (the stage kernels then take over), and several threads at once.

Tolerances: FP64 1e-12 of the largest element over at most 20 steps; FP32
storage 1e-5, its rounding 6e-8 accumulated over 4 x 20 stages."""

import ctypes
import threading

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


def _case(*args):
    print("CASE", *args, flush=True)


# (N, baths, Matsubara terms, depth, complex H): elements per workgroup in the comment
SIZES = [
    (1, 1, 0, 3, False),    # one workgroup, 1 x 1 matrices
    (3, 3, 1, 3, False),    # one workgroup, 747 elements: one per thread
    (4, 4, 0, 4, True),     # one workgroup, 1104 elements: two per thread
    (4, 4, 1, 3, False),    # the smallest grid: 164 workgroups of 16 elements
    (3, 3, 5, 3, False),    # 18 modes: up to 12 "+" entries and 3 "-" ones per element
    (7, 5, 1, 4, True),     # grid, one element per thread
    (14, 7, 0, 5, False),   # 784 elements per workgroup: two per thread
    (16, 16, 0, 3, False),  # 1024: the most for two
    (16, 12, 0, 4, False),  # 2048: the most for four
    (22, 4, 0, 4, False),   # the largest N, 484 elements
]


def _run(prob, steps, dipole, seed):
    N = prob["H"].shape[0]
    obs = {"kind": "population"}
    if dipole:
        obs = {"kind": "dipole", "mu": np.random.default_rng(seed).normal(size=N), "ground": N - 1}
    return dict(prob, dt_fs=0.5, n_steps=steps, record_every=2, observable=obs)


@pytest.mark.parametrize("herm", [True, False])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("size", SIZES, ids=[str(s) for s in SIZES])
def test_resident_run_matches_oracle(heom, orc, size, precision, herm):
    N, nb, M, D, hc = size
    steps = 6
    _case("resident", size, precision, herm)
    run = _run(hi.random_problem(700 + N + D, N, n_baths=nb, M=M, D=D, complex_h=hc), steps, not herm, N)
    if M > 1:
        run["dt_fs"] = 0.05  # the fifth Matsubara rate
    h = heom.Hierarchy(run, precision)
    x = hi.random_state(800 + N, h.n_ado, N, hermitian=herm, scale=0.1)
    if precision == 1:
        x[1:] = x[1:].astype(np.complex64)
    y, rec_ref = orc.propagate(run, x, run["dt_fs"], steps, 2, run["observable"])
    st = h.state_from_numpy(x)
    rec = h.propagate(st, run["dt_fs"], steps, 2, run["observable"], hermitian=herm)
    tol = 1e-12 if precision == 0 else 1e-5
    assert np.max(np.abs(h.state_to_numpy(st) - y)) <= tol * max(1.0, np.max(np.abs(y)))
    assert np.max(np.abs(rec - rec_ref)) <= tol * max(1.0, np.max(np.abs(rec_ref)))


def test_resident_run_longer_than_a_launch(heom):
    """4100 steps are two launches; 4100 calls of one step must agree bit for
    bit in the one-workgroup form, two calls that split the run elsewhere in
    the grid form."""
    for N, M, D, parts in ((2, 0, 3, [1] * 4100), (4, 1, 3, [37, 4063])):
        _case("resident long", N, M, D)
        run = _run(hi.random_problem(31 + N, N, M=M, D=D), 4100, False, 1)
        h = heom.Hierarchy(run, 0)
        a, b = h.new_state(hi.population_rho0(N, 1)), h.new_state(hi.population_rho0(N, 1))
        rec = h.propagate(a, 0.5, 4100, 100, hermitian=True)
        work = h.workspace(4100, 1, 0)
        for k in parts:
            last = h.propagate(b, 0.5, k, k, hermitian=True, work=work)
        assert np.array_equal(h.state_to_numpy(a), h.state_to_numpy(b))
        assert np.array_equal(rec[-1], last[-1])


@pytest.mark.parametrize("precision", [0, 1])
def test_launch_that_gives_up_is_finished_by_stage_kernels(heom, orc, precision):
    """With a zero bound on its waits the grid form gives up; the run is then
    done by the stage kernels from the untouched state."""
    _case("resident fallback", precision)
    lib = heom.load()
    lib.heom_test_resident_wait.argtypes = [ctypes.c_int64]
    lib.heom_test_resident_wait.restype = None
    run = _run(hi.fmo_like(n_steps=12), 12, False, 1)
    h = heom.Hierarchy(run, precision)
    x = hi.random_state(5, h.n_ado, 7, hermitian=True, scale=0.1)
    if precision == 1:
        x[1:] = x[1:].astype(np.complex64)
    y, rec_ref = orc.propagate(run, x, 0.5, 12, 2, run["observable"])
    launches = ctypes.c_int64()
    st = h.state_from_numpy(x)
    lib.heom_test_resident_wait(0)
    lib.heom_timing_enable(1)
    try:
        lib.heom_timing_read(None, None, None, 1)
        rec = h.propagate(st, 0.5, 12, 2, run["observable"], hermitian=True)
        lib.heom_timing_read(None, ctypes.byref(launches), None, 1)
    finally:
        lib.heom_test_resident_wait(-1)
        lib.heom_timing_enable(0)
    tol = 1e-12 if precision == 0 else 1e-5
    assert launches.value == 1 + 4 * 12  # the launch that gave up, then every stage
    assert np.max(np.abs(h.state_to_numpy(st) - y)) <= tol * max(1.0, np.max(np.abs(y)))
    assert np.max(np.abs(rec - rec_ref)) <= tol * max(1.0, np.max(np.abs(rec_ref)))


def test_resident_runs_of_several_threads(heom):
    """Four threads on streams of their own (two grid launches run at a time):
    the same bits as alone."""
    import torch
    _case("resident threads")
    run = _run(hi.fmo_like(n_steps=30), 30, False, 1)
    h = heom.Hierarchy(run, 1)

    def one(seed, stream):
        with torch.cuda.stream(stream):
            st = h.state_from_numpy(hi.random_state(seed, h.n_ado, 7, hermitian=True, scale=0.1))
            work = h.workspace(30, 2, 0)
            stream.synchronize()
            rec = h.propagate(st, 0.5, 30, 2, hermitian=True, work=work, stream=stream)
            stream.synchronize()
        return rec, h.state_to_numpy(st)

    alone = [one(s, torch.cuda.Stream()) for s in range(4)]
    got = [None] * 4
    threads = [threading.Thread(target=lambda s=s: got.__setitem__(s, one(s, torch.cuda.Stream())))
               for s in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, b in zip(alone, got):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def _block_problem(N, M, D, hc, seed):
    """Excited block in its own frame (zero mean energy), three dipole vectors."""
    prob = hi.random_problem(seed, N, M=M, D=D, complex_h=hc)
    prob["H"] = prob["H"] - np.mean(np.diag(prob["H"]).real) * np.eye(N)
    return prob, np.random.default_rng(seed).normal(size=(3, N))


# 60 and 1890 elements, and 62 ADOs whose first has 61 "+" entries, in one
# workgroup; grids of 252, 783 (two per thread) and 1260 (four) per workgroup
@pytest.mark.parametrize("size", [(2, 0, 3, False), (5, 0, 4, False), (1, 60, 1, False),
                                  (7, 1, 4, True), (9, 1, 4, False), (10, 1, 4, False)], ids=str)
def test_resident_block_matches_stages(heom, orc, size):
    """The coherence-block run in one launch gives the bits of the stage
    kernels (a grid that gives up its waits is finished by them); the
    one-workgroup sizes, which wait for nobody, are held to the oracle."""
    N, M, D, hc = size
    _case("resident block", size)
    prob, mu = _block_problem(N, M, D, hc, 900 + N)
    lib = heom.load()
    lib.heom_test_resident_wait.argtypes = [ctypes.c_int64]
    lib.heom_test_resident_wait.restype = None
    dt = 0.005 if M > 1 else 0.5
    h = heom.Hierarchy(prob, 0)
    out = []
    for ticks in (-1, 0):
        y = h.block_state(mu)
        lib.heom_test_resident_wait(ticks)
        try:
            P = h.propagate_block(y, dt, 7, 2, mu)
        finally:
            lib.heom_test_resident_wait(-1)
        out.append((P, y.cpu().numpy()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    if N > 5:
        return
    H = np.zeros((N + 1, N + 1), prob["H"].dtype)
    H[1:, 1:] = prob["H"]
    full = dict(prob, H=H, baths=[dict(b, state=b["state"] + 1) for b in prob["baths"]])
    for p in range(3):
        m = np.concatenate([[0.0], mu[p]])
        rho = np.zeros((N + 1, N + 1), complex)
        rho[:, 0] = m
        y, rec = orc.propagate(full, orc.initial_state(full, h.n_ado, rho), dt, 7, 2,
                               {"kind": "dipole", "mu": m, "ground": 0})
        assert np.max(np.abs(out[0][0][:, p] - (rec[:, 0] + 1j * rec[:, 1]))) <= 1e-12 * np.max(np.abs(rec))
        assert np.max(np.abs(out[0][1][:, :, p] - y[:, 1:, 0])) <= 1e-12 * max(1.0, np.max(np.abs(y)))
