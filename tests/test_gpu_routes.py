"""GPU parity on either side of the lines that the launch code draws between kernels, against the oracle."""
import numpy as np
import pytest

from oracle import dense
from paper_1902_04610_amd import salus, synth
from gpu_util import DevicePool, mlp_layout, norm_rel_err
from test_gpu_kernels import GELU, NONE, RELU, TOL_BF16_TIGHT, run_jobs

pytestmark = pytest.mark.gpu


def check(specs, launches):
    outs, refs, n = run_jobs(specs, salus.BF16)
    assert n == launches
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all(), j
        assert norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))


@pytest.mark.parametrize("jobs, M, K, N, strip", [
    (1, 129, 200, 8, False), (7, 192, 1096, 520, False),                 # register tiles
    (16, 255, 520, 512, True),                                           # 512 of them: the last round that takes them
    (17, 255, 520, 512, True), (12, 385, 1096, 520, False),              # the tiled kernel
    (6, 300, 2056, 776, False), (5, 300, 2056, 776, False),              # deep: 420 / 350 register tiles, both tiled
    (4, 300, 2056, 776, False),                                          # 280: register tiles
    (40, 200, 72, 1032, False),                                          # fewer than three slabs: never tiled
])
def test_ragged_depth_above_128_rows(jobs, M, K, N, strip):
    check([dict(M=max(129, M - 13 * (i % 6)), dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)], 1)


def test_a_row_of_infinities_stays_in_its_row_of_a_large_tile():
    """Enough jobs for the tiled kernel; the contraction (200) ends inside a slab: neither the next row of X nor what follows W
    reaches the sums."""
    jobs, M, K, N = 26, 200, 200, 264
    w_offs, P, x_off, y_off, h_off, E = mlp_layout((K, N), 2, M)
    dp = DevicePool(jobs * (P + 4096 + E), policy=salus.POLICY_PACK)
    rng = np.random.default_rng(3)
    W = synth.f32_to_bf16_bits((rng.standard_normal((K, N)) / np.sqrt(K)).astype(np.float32))
    X = synth.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    ref = dense.mlp_forward_bf16(X, [W], [NONE])[-1]
    X[7] = 0x7f80                                                  # a row of +inf; row 6 ends where it begins
    items, lanes = [], []
    for _ in range(jobs):
        st, job = dp.pool.lane_alloc(P + 4096, E, 0, 1)
        assert st == salus.OK
        q = dp.pool.job_query(job)
        dp.write(q.persist_off, W)
        dp.write(q.persist_off + W.nbytes, np.full(4096 // 2, 0x7fc0, np.uint16))      # NaN right behind the weights
        dp.write(q.lane_off + x_off, X)
        items.append(dict(job=job, M=M, dtype=salus.BF16, layers=[(K, N, 0, NONE)], x_off=x_off, y_off=y_off, h_off=h_off))
        lanes.append(q.lane_off)
    descs, keep = salus.Pool.make_descs(items)
    assert dp.pool.grouped_forward(descs, stream=dp.stream) == salus.OK
    dp.sync()
    rows = np.arange(M) != 7
    for lane in lanes:
        Y = dp.read(lane + y_off, M * N * 4, np.float32).reshape(M, N)
        assert not np.isfinite(Y[7]).any()
        assert norm_rel_err(Y[rows], ref[rows]) < TOL_BF16_TIGHT
    dp.close()
