"""In which order the LDS-tiled kernels add the products of an output: where a job is computed changes nothing that it did not change before."""
import numpy as np
import pytest

from gpu_util import DevicePool, mlp_layout
from paper_1902_04610_amd import salus, synth

pytestmark = pytest.mark.gpu


def forward(jobs):
    """One round of single layers without activation; jobs: (X, W) as bf16 bits."""
    layouts = [mlp_layout((X.shape[1], W.shape[1]), 2, X.shape[0]) for X, W in jobs]
    dp = DevicePool(sum(t[1] + t[5] for t in layouts) + 4096, policy=salus.POLICY_PACK)
    items, at = [], []
    for (X, W), (_, P, x_off, y_off, h_off, E) in zip(jobs, layouts):
        st, job = dp.pool.lane_alloc(P, E, 0, 1)
        assert st == salus.OK
        q = dp.pool.job_query(job)
        dp.write(q.persist_off, W)
        dp.write(q.lane_off + x_off, X)
        items.append(dict(job=job, M=X.shape[0], dtype=salus.BF16, layers=[(*W.shape, 0, salus.ACT_NONE)], x_off=x_off, y_off=y_off, h_off=h_off))
        at.append(q.lane_off + y_off)
    descs, keep = salus.Pool.make_descs(items)
    assert dp.pool.grouped_forward(descs, stream=dp.stream) == salus.OK, dp.pool.last_error()
    dp.sync()
    out = [dp.read(a, X.shape[0] * W.shape[1] * 4, np.float32).reshape(X.shape[0], W.shape[1]).copy() for a, (X, W) in zip(at, jobs)]
    dp.close()
    return out


@pytest.mark.parametrize("jobs, M, N, slabs", [(17, 33, 512, 2), (24, 64, 520, 5)])
def test_64_by_64_tiles_of_the_ring_keep_two_sums(jobs, M, N, slabs):
    """One over the first half of every slab of 64, one over the second: 2^24 and its negative in a first half take nothing from ones in second
    halves, which a single sum in order of k would round away."""
    X = np.zeros((M, 64 * slabs), np.float32)
    X[:, 0], X[:, 64 * (slabs - 1)] = 2.0 ** 24, -2.0 ** 24
    X[:, 32::64] = 1.0
    job = synth.f32_to_bf16_bits(X), synth.f32_to_bf16_bits(np.ones((64 * slabs, N), np.float32))
    for Y in forward([job] * jobs):
        assert (Y == slabs).all()


@pytest.mark.parametrize("rows, K, N", [([129, 193], 448, 2056), ([256] * 4, 384, 1024), ([200] * 5, 448, 1096), ([268] * 5, 512, 2392)])
def test_few_jobs_of_128_rows_and_more_have_the_bits_that_large_tiles_give(rows, K, N):
    """64 x 64 and 64 x 128 ring tiles; beside more jobs the same ones take tiles of 128 rows and more."""
    rng = np.random.default_rng(K)
    bits = lambda *shape: synth.f32_to_bf16_bits(rng.standard_normal(shape).astype(np.float32))
    jobs = [(bits(m, K), bits(K, N)) for m in rows]
    few = forward(jobs)
    many = forward(jobs + [(bits(300, K), jobs[0][1])] * 40)
    for a, b in zip(few, many):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
