"""GPU parity of launches on either side of eight problems, where the arguments that a kernel is passed change, against the oracle."""
import numpy as np
import pytest

from gpu_util import norm_rel_err
from paper_1902_04610_amd import salus
from test_gpu_kernels import GELU, NONE, RELU, TOL_BF16_TIGHT, TOL_F32, run_jobs

pytestmark = pytest.mark.gpu

# type, rows of the first job, layers, kernels; every kernel that has both kinds of arguments in one of them
EDGE = [
    ("bf16", 1, (1000, 520, 72), ["bf16_narrow<1, false, 2, 0, true>", "bf16_narrow<1, false, 1, 0, true>"]),
    ("bf16", 17, (264, 136), ["bf16_narrow<2, false, 1, 0, true>"]), ("bf16", 8, (520, 1544), ["bf16_narrow<1, false, 4, 0, true>"]),
    ("bf16", 32, (520, 776, 1544), ["bf16_narrow<2, false, 2, 0, true>", "bf16_narrow<2, false, 4, 0, true>"]),
    ("bf16", 36, (264, 136, 1032), ["bf16_narrow<2, false, 2, 8, false>", "bf16_stream<64, 64, 2, 1, 2, false, 4>"]),
    ("bf16", 140, (448, 136), ["bf16_narrow<2, false, 2, 8, false>"]), ("bf16", 64, (264, 776), ["bf16_narrow<2, false, 4, 4, false>"]),
    ("f32", 8, (260, 132), ["f32_narrow"]), ("f32", 30, (132, 900), ["f32<1>"]), ("f32", 60, (516, 516), ["f32<2>"]),
    ("f32", 129, (132, 1028), ["f32<4>"]), ("f32", 12, (276, 1204), ["f32<1>"]),
]


@pytest.mark.parametrize("jobs", [8, 9])
@pytest.mark.parametrize("dtype, M, dims, kernels", EDGE)
def test_eight_and_nine_problems(dtype, M, dims, kernels, jobs):
    f32 = dtype == "f32"
    specs = [dict(M=M - (i % 3 if M > 3 else 0), dims=dims, acts=([GELU, RELU] * 2)[i % 2:][:len(dims) - 2] + [NONE]) for i in range(jobs)]
    outs, refs, launches = run_jobs(specs, salus.F32 if f32 else salus.BF16)
    assert launches == len(dims) - 1
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < (TOL_F32 if f32 else TOL_BF16_TIGHT), (j, norm_rel_err(o, r))
