"""GPU parity of launches whose weights are asked for once, from further away than the memory-side cache, against the oracle."""
import numpy as np
import pytest

import test_gpu_kernels
from gpu_util import DevicePool, norm_rel_err
from paper_1902_04610_amd import salus
from test_gpu_kernels import GELU, NONE, RELU, TOL_BF16_TIGHT, run_jobs

pytestmark = pytest.mark.gpu


class FarPool(DevicePool):
    """A pool that holds 240 MB of another job's state besides."""

    def __init__(self, capacity, **kw):
        idle = 240 << 20
        super().__init__(capacity + idle + 4096, **kw)
        assert self.pool.lane_alloc(idle, 256, 0, 0)[0] == salus.OK


# jobs, largest rows, K, N, strips; the kernel of the launch
ONCE = [
    (64, 128, 320, 1000, False), (60, 90, 1032, 1288, False), (65, 70, 320, 1024, True), (48, 128, 1096, 1544, False),
]


@pytest.mark.parametrize("jobs, M, K, N, strip", ONCE)
def test_weights_asked_for_once(jobs, M, K, N, strip, monkeypatch):
    """Tiles that end inside the matrices, depths of less than the ring and no multiple of a slab, more jobs than a launch holds."""
    monkeypatch.setattr(test_gpu_kernels, "DevicePool", FarPool)
    specs = [dict(M=M - (i % 3) * 2, dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)]
    outs, refs, _ = run_jobs(specs, salus.BF16)
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all(), j
        assert norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))
