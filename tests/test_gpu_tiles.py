"""GPU parity of the LDS-tiled kernels at the edges of their tiles, slabs and dispatch rule, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import dense
from paper_1902_04610_amd import salus, synth
from gpu_util import DevicePool, mlp_layout, norm_rel_err
from test_gpu_kernels import GELU, NONE, RELU, TOL_BF16_TIGHT, TOL_F32, run_jobs
from test_gpu_train import run as run_training

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("jobs, M, K, N, strip", [
    (20, 250, 200, 4104, False),      # 340 tiles of 256 x 256: workgroups walk two, the request stream crosses tile ends
    (16, 193, 256, 4096, True),       # as many tiles as compute units
    (8, 257, 264, 4096, False),       # 128 x 256
    (33, 128, 64, 2176, True),        # 128 x 256 / 128 x 128, one slab of data in three
    (1, 192, 192, 8, False), (1, 1024, 448, 136, False), (2, 385, 1096, 520, False),       # 128 x 128, tails everywhere
    (80, 200, 128, 1032, False),      # 128 x 128 x 2 per compute unit or larger tiles, more than 64 problems
])
def test_tile_kinds_and_tails(jobs, M, K, N, strip):
    specs = [dict(M=M - (i % 3 if M > 192 else 0), dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)]
    outs, refs, _ = run_jobs(specs, salus.BF16)
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all(), j
        assert norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))


def test_a_row_of_infinities_stays_in_its_row():
    """The contraction (200) ends inside a slab: what is fetched beyond it - the next row of X, whatever follows W -
    must not reach the sums, infinite or not."""
    M, K, N = 200, 200, 264
    dp = DevicePool(1 << 20, policy=salus.POLICY_PACK)
    w_offs, P, x_off, y_off, h_off, E = mlp_layout((K, N), 2, M)
    rng = np.random.default_rng(3)
    W = synth.f32_to_bf16_bits((rng.standard_normal((K, N)) / np.sqrt(K)).astype(np.float32))
    X = synth.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    ref = dense.mlp_forward_bf16(X, [W], [NONE])[-1]
    X[7] = 0x7f80                                                  # a row of +inf; row 6 ends where it begins
    st, job = dp.pool.lane_alloc(P + 4096, E, 0, 1)
    q = dp.pool.job_query(job)
    dp.write(q.persist_off, W)
    dp.write(q.persist_off + W.nbytes, np.full(4096 // 2, 0x7fc0, np.uint16))      # NaN right behind the weights
    dp.write(q.lane_off + x_off, X)
    descs, keep = salus.Pool.make_descs([dict(job=job, M=M, dtype=salus.BF16, layers=[(K, N, 0, NONE)], x_off=x_off,
                                              y_off=y_off, h_off=h_off)])
    assert dp.pool.grouped_forward(descs, stream=dp.stream) == salus.OK
    dp.sync()
    Y = dp.read(q.lane_off + y_off, M * N * 4, np.float32).reshape(M, N)
    rows = np.arange(M) != 7
    assert not np.isfinite(Y[7]).any()
    assert norm_rel_err(Y[rows], ref[rows]) < TOL_BF16_TIGHT
    dp.close()


@pytest.mark.parametrize("jobs, M, K, N, strip", [
    (1, 33, 8, 8, False), (2, 64, 72, 128, True), (3, 65, 1096, 264, False), (1, 128, 520, 1024, True),
    (4, 50, 256, 384, True),          # 64 x 64 tiles: some begin in the middle of a strip of 128 columns
    (40, 100, 72, 1032, False),       # 64 x 128 tiles, 720 of them: workgroups walk two, fewer slabs than the ring has stages
    (30, 128, 264, 1152, True),
    (36, 70, 1032, 2056, False),      # deep, more than 64 rows, fills the chip: the compute-bound kernel takes them all
    (16, 66, 1096, 1544, False),      # 112 tiles of 128 x 256, not enough to fill the chip: the same
    (30, 87, 1096, 768, True),        # 90: one launch through the ring, of jobs on either side of 64 rows
    (13, 64, 1032, 1288, False),      # 64 x 64 tiles would be 273, more than one per compute unit: 64 x 128
])
def test_rows_33_to_128_through_the_ring(jobs, M, K, N, strip):
    specs = [dict(M=max(33, M - (i % 5) * 7), dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)]
    outs, refs, launches = run_jobs(specs, salus.BF16)
    assert launches == 1
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all(), j
        assert norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))


@pytest.mark.parametrize("dims, M", [((72, 136, 8), 33), ((520, 264, 40), 64), ((264, 1032, 72), 130), ((192, 200, 1000), 300)])
def test_input_gradients_through_the_ring(dims, M):
    """The transposed product, masked by the ReLU derivative, at ragged widths."""
    run_training([(dims, M, 0.05)], steps=1, seed=4)


@pytest.mark.parametrize("configs", [
    [((136, 520, 40), 257, 0.05)], [((64, 72), 256, 0.05), ((264, 128, 136), 333, 0.01)],
    [((200, 1096, 264), 600, 0.02)],          # several slabs of batch, more tiles than compute units would need
    [((72, 40), 16, 0.1), ((72, 40), 17, 0.1), ((40, 1032), 18, 0.1)],      # rows of one and of two workgroups of the loss
])
def test_updates_of_many_rows_and_loss_rows(configs):
    """The weight gradient through the LDS tiles (256 rows on average and more), and jobs around the loss kernel's 16 rows."""
    run_training(configs, steps=2, seed=12)


@pytest.mark.parametrize("configs", [[((136, 264, 72), 191, 0.05)], [((136, 264, 72), 192, 0.05)], [((2056, 4232), 193, 0.05)]])
def test_updates_around_192_rows(configs):
    """The register kernel below 192 rows, LDS tiles from there; the last one has more tiles than workgroups: master weights of the
    next tile are requested while those of the last are stored."""
    run_training(configs, steps=1, seed=13)


@pytest.mark.parametrize("shift_mb, blocks", [(79, 3), (80, 3), (81, 2), (96, 4)])
def test_equal_shifts_move_as_one(shift_mb, blocks):
    """All blocks above the only hole move by its size: one move, in place below 80 MiB and in pieces of the shift
    from there on (the last piece is a remainder)."""
    MiB = 1 << 20
    sizes = [shift_mb * MiB] + [90 * MiB + 4096 * (i + 1) for i in range(blocks)]
    dp = DevicePool(sum(sizes) + 16 * MiB, max_lanes=1)
    scratch = torch.zeros(8, dtype=torch.uint8, device="cuda")
    for i, s in enumerate(sizes):
        st, job = dp.pool.lane_alloc(s, 4096, 0, 1)
        assert st == salus.OK
        salus.fill_pattern(dp.buf.data_ptr() + dp.pool.job_query(job).persist_off, s, 100 + i)
    for again in range(2):                        # the counters of the in-place kernel run on from move to move
        assert dp.pool.lane_free(again) == salus.OK
        plan = dp.pool.compact()
        assert len(plan) == len(sizes) - 1 - again and len({src - dst for src, dst, _ in plan}) == 1
        for i in range(again + 1, len(sizes)):
            q = dp.pool.job_query(i)
            assert q.persist_off == sum(sizes[again + 1:i])
            assert salus.check_pattern(dp.buf.data_ptr() + q.persist_off, sizes[i], 100 + i, scratch.data_ptr()) == 0
    dp.close()


@pytest.mark.parametrize("M", [1, 16, 17, 32])
@pytest.mark.parametrize("copies", [1, 9, 17])
def test_few_jobs_take_narrow_tiles(M, copies):
    """1, 9, 17 copies of three shapes: 32-, 64- and 128-column tiles in the wider layers."""
    shapes = [((8, 8), False), ((2120, 1000), False), ((136, 512, 384, 72), True)]
    specs = [dict(M=M, dims=d, acts=[GELU] * (len(d) - 2) + [RELU], strip=s) for d, s in shapes]
    outs, refs, _ = run_jobs(specs * copies, salus.BF16)
    for o, r, j in zip(outs, refs, specs * copies):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))


@pytest.mark.parametrize("configs", [[((136, 520, 264, 72), 20, 0.05)], [((264, 1032, 72), 24, 0.05)] * 9, [((2104, 136, 40), 9, 0.05)]])
def test_input_gradients_of_few_rows(configs):
    """Narrow tiles of the transposed product, and the ring from 17 rows with enough jobs."""
    run_training(configs, steps=1, seed=5)


@pytest.mark.parametrize("jobs, M", [(1, 16), (1, 17), (3, 64), (3, 65), (40, 33), (40, 66), (2, 200)])
def test_float_row_tiles(jobs, M):
    """16-, 32- and 64-row tiles, and last tiles that compute only the 16-row blocks they need."""
    specs = [dict(M=max(1, M - 15 * (i % 4)), dims=(132, 68 + 260 * (i % 3), 64), acts=[GELU, RELU]) for i in range(jobs)]
    outs, refs, _ = run_jobs(specs, salus.F32)
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_F32, (j, norm_rel_err(o, r))


# jobs, rows, K, N, strips; every tile of 128 x 128
TAILS = [(12, 257, 448, 1032, False), (9, 385, 1096, 520, False), (5, 500, 448, 1288, False), (3, 513, 448, 2688, True)]


@pytest.mark.parametrize("jobs, M, K, N, strip", TAILS)
def test_tails_of_128_by_128_tiles(jobs, M, K, N, strip):
    """Deeper than the ring, rows and columns that end inside a tile, one or two tiles per compute unit."""
    specs = [dict(M=M - (i % 3), dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)]
    outs, refs, _ = run_jobs(specs, salus.BF16)
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))


# jobs, layers, rows, columns of the ring's tiles
RING_GRADIENTS = [
    (17, (72, 520, 264), 33, 64), (4, (264, 1032, 136), 70, 64), (4, (136, 1544, 264), 129, 64), (2, (40, 1032, 1000), 300, 64),
    (30, (72, 1032, 264), 50, 128), (7, (72, 1032, 72), 257, 128),
]


@pytest.mark.parametrize("jobs, dims, M, columns", RING_GRADIENTS)
def test_input_gradients_of_many_tiles_through_the_ring(jobs, dims, M, columns):
    """64 x 64 tiles, whose wavefronts store masked half lines, and 64 x 128; depths and widths that end inside a slab, a line and a tile."""
    run_training([(dims, M, 0.05)] * jobs, steps=1, seed=14)
