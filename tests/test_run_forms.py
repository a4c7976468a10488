"""How runs are done, on the host: the kernel at both sides of the bounds."""

import numpy as np
import pytest

import run_forms as rf

FP64, FP32, HERM = 0, 1, 2


def _prob(N, nb, M, D):
    return {"H": np.zeros((N, N)), "temperature_K": 300.0, "depth": D, "flags": 0,
            "baths": [{"state": s, "lambda_cm": 35.0, "tau_fs": 50.0, "matsubara": M} for s in range(nb)]}


@pytest.mark.parametrize("precision, N, nb, M, D, kernel", [
    # deep FP32 hierarchies of one mode per state: the "+" sums outweigh the bytes
    (FP32, 26, 8, 0, 8, "k_stage_persist"),
    (FP32, 28, 9, 0, 7, "k_stage_persist"),
    (FP32, 22, 11, 0, 7, "k_stage_persist"),
    (FP32, 30, 10, 0, 8, "k_stage_persist"),
    # several modes per state, and odd N: from 10 million elements
    (FP32, 22, 5, 1, 7, "k_stage_persist"),
    (FP32, 24, 5, 1, 7, "k_packed"),
    (FP32, 27, 9, 0, 7, "k_stage_persist"),
    (FP32, 25, 12, 0, 6, "k_packed"),
    # not deep, or of other sizes: as before
    (FP32, 24, 24, 0, 4, "k_packed"),
    (FP32, 17, 17, 0, 5, "k_packed"),
    (FP32, 32, 10, 0, 6, "k_packed"),
    (FP32, 33, 33, 0, 3, "k_packed"),
    (FP32, 48, 48, 1, 3, "k_packed"),
    # packed storage with three row blocks
    (HERM, 44, 14, 2, 2, "k_bulk_mfma_pk"),
    (HERM, 44, 44, 0, 2, "k_bulk_mfma_pk"),
    (HERM, 48, 16, 0, 3, "k_packed"),
    (HERM, 30, 30, 1, 2, "k_packed"),
    (HERM, 52, 17, 1, 2, "k_packed"),
    (HERM, 33, 33, 1, 3, "k_packed"),
    (FP64, 26, 8, 0, 7, "k_packed"),
    (FP64, 48, 48, 1, 3, "k_packed"),
    # one column per lane: the tiles outweigh the "+" links below the top level
    (FP32, 7, 3, 20, 3, "k_stage_small"),
    (FP32, 5, 5, 20, 3, "k_stage_small"),
    (FP32, 6, 6, 20, 3, "k_stage_small"),
    (FP32, 6, 6, 4, 4, "k_stage_small"),
    (FP32, 5, 5, 2, 8, "k_columns"),
    (FP32, 7, 7, 5, 6, "k_columns"),
    (FP32, 5, 5, 30, 3, "k_columns"),
    (FP64, 4, 4, 14, 3, "k_stage_small"),
    (FP64, 5, 5, 20, 3, "k_stage_small"),
    (FP64, 2, 2, 20, 4, "k_columns"),
    (FP64, 6, 3, 30, 3, "k_columns"),
    (FP64, 7, 7, 5, 6, "k_columns"),
])
def test_kernel_where_it_pays(precision, N, nb, M, D, kernel):
    assert rf.run_kernel(_prob(N, nb, M, D), precision) == kernel


def test_bench_names_the_kernel_that_runs():
    """Sizes that one launch could hold by their elements, and does not by its
    LDS (16 states, 1820 ADOs) or for its workspace (495 ADOs of 2 x 2 in FP32)."""
    import bench
    import paper_1803_03498_amd as heom
    assert bench._bulk_kernel_name(_prob(16, 12, 0, 4), FP64, heom) == "k_bulk_mfma"
    assert bench._bulk_kernel_name(_prob(16, 12, 0, 4), FP32, heom) == "k_resident"
    assert bench._bulk_kernel_name(_prob(2, 2, 1, 8), FP32, heom) == "k_bulk_fma"
    assert bench._bulk_kernel_name(_prob(24, 3, 2, 10), FP64, heom) == "k_bulk_mfma"  # depth above the modes
