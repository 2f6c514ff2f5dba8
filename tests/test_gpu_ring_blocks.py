"""GPU parity of bf16 results of 64 x 64 tiles, whose wavefronts store half lines, at widths that end inside one, against the oracle."""
import numpy as np
import pytest

from gpu_util import norm_rel_err
from paper_1902_04610_amd import salus
from test_gpu_kernels import GELU, NONE, RELU, TOL_BF16_TIGHT, run_jobs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("jobs, dims, M", [
    (24, (136, 520, 72), 33), (20, (72, 536, 40), 64), (12, (264, 1000, 24), 65), (7, (200, 1064, 136), 127),
])
def test_hidden_activations_in_half_lines(jobs, dims, M):
    specs = [dict(M=max(33, M - 5 * (i % 4)), dims=dims, acts=[[GELU, RELU, NONE][i % 3], NONE]) for i in range(jobs)]
    outs, refs, _ = run_jobs(specs, salus.BF16)
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))
