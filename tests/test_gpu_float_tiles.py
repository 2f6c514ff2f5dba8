"""GPU parity of float layers on either side of the line between 16- and 32-row tiles, against the oracle and the depth-fused launch."""
import numpy as np
import pytest

from gpu_util import norm_rel_err
from paper_1902_04610_amd import salus
from test_gpu_kernels import GELU, NONE, TOL_F32, run_jobs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows, dims", [
    ([1, 9, 16, 17, 31, 33, 48, 49, 64, 80], (268, 900, 60)), ([95] * 5, (260, 696, 12)), ([33] * 9, (300, 708, 12)), ([16] * 20, (44, 1028, 8)),
])
def test_float_rows_on_both_sides(rows, dims):
    specs = [dict(M=m, dims=dims, acts=[GELU, NONE]) for m in rows]
    outs, refs, _ = run_jobs(specs, salus.F32)
    fused, _, _ = run_jobs(specs, salus.F32, fuse=True)
    for o, r, f, j in zip(outs, refs, fused, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_F32, (j, norm_rel_err(o, r))
        assert np.array_equal(o.view(np.uint32), f.view(np.uint32)), j


@pytest.mark.parametrize("rows, dims", [([16] * 12, (260, 1204)), ([1, 15, 16, 17] * 5, (320, 700)), ([2] * 82, (276, 944)), ([7, 16] * 6, (300, 1204, 512, 12)), ([9] * 30, (452, 516)), ([5] * 16, (1068, 1380, 8))])
def test_float_layers_with_four_steps_in_flight(rows, dims):
    specs = [dict(M=m, dims=dims, acts=[GELU] * (len(dims) - 2) + [NONE]) for m in rows]
    outs, refs, _ = run_jobs(specs, salus.F32)
    fused, _, _ = run_jobs(specs, salus.F32, fuse=True)
    for o, r, f, j in zip(outs, refs, fused, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_F32, (j, norm_rel_err(o, r))
        assert np.array_equal(o.view(np.uint32), f.view(np.uint32)), j
