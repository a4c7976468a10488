"""Resident runs (one launch for a whole run) inside the caller's workspace, on
the host: over every size the plan takes, the flags and stage copies of the
launches end in front of the records."""

import ctypes
from math import comb

import numpy as np
import pytest

import heom_inputs as hi


@pytest.fixture(scope="module")
def plan():
    import paper_1803_03498_amd as heom
    lib = heom.load()
    lib.heom_test_resident_plan.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.POINTER(ctypes.c_size_t)]
    lib.heom_test_resident_plan.restype = ctypes.c_int32

    def call(prob, precision, herm=True):
        p = heom.Problem(prob, precision)
        out = (ctypes.c_size_t * 4)()
        route = lib.heom_test_resident_plan(ctypes.byref(p.struct), 1 if herm else 0, out)
        assert route >= 0
        return route, list(out), heom.plan(p)

    return call


def _sizes():
    """(N, W, D) whose ADOs a resident run could hold: at most 255 workgroups
    of 2048 elements."""
    for N in range(1, 23):
        for D in range(1, 255):
            for W in range(1, 256 - D):
                if (comb(W + D, W) - 1) * N * N > 255 * 2048:
                    break
                yield N, W, D


def test_launches_stay_in_front_of_the_records(plan):
    up = lambda x: (x + 255) // 256 * 256
    grids, refused = 0, 0
    for N, W, D in _sizes():
        prob = {"H": np.zeros((N, N)), "temperature_K": 300.0, "depth": D, "flags": 0,
                "baths": [{"state": 0, "lambda_cm": 35.0, "tau_fs": 50.0, "matsubara": W - 1}]}
        for precision in (0, 1):
            route, (end, have, _, groups), info = plan(prob, precision)
            if route != 2:
                refused += route == 0
                continue
            grids += 1
            need = 1024 + up(8 * N) + up(64 * groups) + 2 * up(info["sigma0_bytes"]) + 2 * up(info["rest_bytes"])
            assert have == info["work_bytes"]
            assert need <= end <= have, (N, W, D, precision)
    assert grids > 1000 and refused > 0


def test_small_grids_keep_their_form(plan):
    """Sizes whose flags for 256 workgroups would not fit but whose own do; one
    that has room for neither runs stage by stage."""
    for N, nb, M, D, precision, route in ((12, 12, 0, 1, 1, 2), (20, 3, 0, 1, 1, 2), (3, 3, 2, 3, 1, 2),
                                          (2, 2, 0, 16, 0, 2), (2, 2, 1, 8, 1, 0)):
        assert plan(hi.random_problem(1, N, n_baths=nb, M=M, D=D), precision)[0] == route, (N, nb, M, D)


def test_two_grid_launches_fit_the_gpu(plan):
    """Two workgroups fit a CU's 160 KiB of LDS, the launch's static word (16
    bytes with its alignment) included: two launches can be on the GPU together."""
    most = 0
    for N, W, D in _sizes():
        prob = {"H": np.zeros((N, N)), "temperature_K": 300.0, "depth": D, "flags": 0,
                "baths": [{"state": s % N, "lambda_cm": 35.0, "tau_fs": 50.0, "matsubara": 0} for s in range(W)]}
        for precision in (0, 1):
            for herm in ((True, False) if precision == 0 else (True,)):
                route, (_, _, lds, groups), _ = plan(prob, precision, herm)
                if route == 2:
                    most = max(most, lds)
                    assert 2 * (lds + 16) <= 160 * 1024, (N, W, D, precision, herm)
                    assert groups <= 256
    assert most > 78 * 1024  # the bound is reached
