"""GPU parity of jobs of 128 rows and more that are too few for large tiles, at the edges of the tiles that they take, against the oracle."""
import numpy as np
import pytest

from gpu_util import norm_rel_err
from paper_1902_04610_amd import salus
from test_gpu_kernels import GELU, NONE, RELU, TOL_BF16_TIGHT, run_jobs

pytestmark = pytest.mark.gpu

# rows, K, N, strips, the launch of the layer
FEW = [
    ([128], 384, 8, False, "narrow<2, false, 2, 8, false>"), ([129, 160, 500], 448, 264, False, "narrow<2, false, 2, 8, false>"),
    ([255], 2112, 1024, True, "narrow<2, false, 2, 8, false>"), ([257], 384, 1024, True, "narrow<2, false, 4, 4, false>"),
    ([130, 300], 576, 1000, False, "narrow<2, false, 4, 4, false>"),
    ([129, 193], 448, 2056, False, "stream<64, 64, 2, 1, 2, false, 4>"), ([256] * 4, 384, 1024, True, "stream<64, 64, 2, 1, 2, false, 4>"),
    ([200] * 5, 448, 1096, False, "stream<64, 128, 2, 2, 2, false, 3>"), ([512] * 2, 384, 2048, True, "stream<64, 128, 2, 2, 2, false, 3>"),
    ([268] * 5, 512, 2392, False, "stream<64, 128, 2, 2, 1, false, 3>"), ([200] * 5, 2120, 1288, False, "stream<64, 128, 2, 2, 2, false, 3>"),
]


@pytest.mark.parametrize("rows, K, N, strip, kernel", FEW)
def test_few_tiles(rows, K, N, strip, kernel):
    """Two layers, so that results are stored as bf16 and as float."""
    specs = [dict(M=m, dims=(K, N, 72), acts=[[GELU, RELU, NONE][i % 3], NONE], strip=strip) for i, m in enumerate(rows)]
    outs, refs, _ = run_jobs(specs, salus.BF16)
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))
