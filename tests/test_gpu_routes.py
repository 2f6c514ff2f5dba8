"""GPU parity on either side of the lines that the launch code draws between kernels, against the oracle."""
import numpy as np
import pytest

from oracle import dense
from paper_1902_04610_amd import salus, synth
from gpu_util import DevicePool, mlp_layout, norm_rel_err
from test_gpu_kernels import GELU, NONE, RELU, TOL_BF16_TIGHT, TOL_F32, run_jobs

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


@pytest.mark.parametrize("jobs, M, K, N, strip", [
    (1, 33, 8, 8, False), (1, 128, 2056, 264, False), (3, 65, 1096, 264, True), (4, 64, 136, 1024, True),       # 32 columns, the last two to the tile
    (1, 97, 2056, 2056, False), (16, 64, 128, 512, True), (3, 50, 520, 2056, False),        # 64 columns, deep and not
    (17, 64, 128, 512, True), (8, 128, 264, 520, False), (16, 40, 72, 1000, False), (70, 33, 200, 136, False),       # the ring, 64 x 64 tiles
    (9, 128, 72, 1032, True),                                                                # the ring, 64 x 128
])
def test_rows_33_to_128_around_the_ring(jobs, M, K, N, strip):
    """Rows of a job's second tile read the same weights; some tiles begin in the middle of a strip of 128 columns."""
    check([dict(M=max(33, M - 7 * (i % 4)), dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)],
          1 if jobs <= 64 else 2)


def test_hidden_layers_of_33_to_128_rows_in_narrow_tiles():
    """bf16 hidden activations, written and read by narrow tiles."""
    check([dict(M=m, dims=(136, 264, 72, 520), acts=[GELU, RELU, NONE], strip=False) for m in (33, 63, 64, 90, 127)], 3)


@pytest.mark.parametrize("jobs, M, K, N", [(12, 32, 516, 780), (12, 32, 132, 780), (60, 17, 68, 388), (26, 40, 1028, 964), (17, 64, 1032, 1536)])
def test_float_rows_around_the_lines(jobs, M, K, N):
    """32-row tiles of 17 .. 32 rows, and 64-row tiles of deep layers that fill the chip with one each."""
    specs = [dict(M=max(17 if M <= 32 else 33, M - 5 * (i % 3)), dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]]) for i in range(jobs)]
    outs, refs, n = run_jobs(specs, salus.F32)
    assert n == 1
    for o, r, j in zip(outs, refs, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_F32, (j, norm_rel_err(o, r))


@pytest.mark.parametrize("jobs, M, K, N, strip, launches", [
    (2, 300, 64, 1024, True, 1), (8, 160, 128, 1032, False, 1), (1, 700, 256, 2056, False, 1),      # register tiles
    (3, 128, 64, 1024, False, 1),                                        # 128 rows: the narrow tiles of fewer rows
    (40, 200, 64, 1024, True, 1), (6, 700, 256, 2056, False, 1),         # tiled: float rows that begin on a line and that do not
])
def test_shallow_depth_from_128_rows(jobs, M, K, N, strip, launches):
    check([dict(M=M, dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)], launches)


@pytest.mark.parametrize("jobs, M, K, N", [(20, 250, 320, 4096), (70, 256, 320, 4096), (40, 40, 520, 4096), (3, 300, 576, 520)])
def test_float_outputs_past_l2(jobs, M, K, N):
    """Results stored past L2 (rows that begin on a line; 256 x 256 tiles below one round and above three) and not."""
    check([dict(M=M - (i % 2), dims=(K, N), acts=[[GELU, RELU, NONE][i % 3]], strip=False) for i in range(jobs)], 1 if jobs <= 64 else 2)


@pytest.mark.parametrize("jobs, M, Ks, N, strip", [
    (64, 65, [320], 1024, True),                    # one tile for every workgroup
    (33, 300, [320, 320, 328], 1544, False),        # more tiles than workgroups, the walk crosses from one depth to another
    (33, 299, [448, 320], 1024, True), (64, 100, [384], 1544, False),
])
def test_two_tiles_of_128_by_256_per_compute_unit(jobs, M, Ks, N, strip):
    check([dict(M=max(65, M - 7 * (i % 3)), dims=(Ks[i % len(Ks)], N), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)], 1)


def test_hidden_layers_in_two_tiles_of_128_by_256_per_compute_unit():
    """bf16 outputs of such tiles, and their use as inputs; rows end inside a tile."""
    check([dict(M=293 + i % 8, dims=(328, 1544, 136), acts=[GELU if i % 2 else RELU, NONE], strip=False) for i in range(33)], 2)


@pytest.mark.parametrize("jobs, dims, strip", [
    (1, (8, 8), False), (1, (24, 16, 40, 8), False), (3, (4104, 24), False), (2, (1000, 2056, 264, 520), False), (2, (512, 1024, 128), True),      # 16 columns
    (5, (264, 1032, 136), False), (7, (1032, 1024, 32), True),                               # 32 (layers of 1024 columns)
    (12, (520, 1032, 8), False), (14, (136, 1024, 1032), True),                              # 64
])
def test_narrow_tiles_up_to_32_rows(jobs, dims, strip):
    """Depths that end inside a k-step, a pair of them or the ring; widths that end inside a tile; 1 - 32 rows, one row tile and two
    in a launch.  The order of the sums is that of the wide tiles: the depth-fused launch gives the same bits."""
    specs = [dict(M=[1, 16, 17, 32, 7][i % 5], dims=dims, acts=([GELU, RELU] * 2)[:len(dims) - 2] + [NONE], strip=strip) for i in range(jobs)]
    outs, refs, n = run_jobs(specs, salus.BF16)
    assert n == len(dims) - 1
    fused, _, _ = run_jobs(specs, salus.BF16, fuse=True)
    for o, r, f, j in zip(outs, refs, fused, specs):
        assert np.isfinite(o).all(), j
        assert norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))
        assert np.array_equal(o.view(np.uint32), f.view(np.uint32)), j


@pytest.mark.parametrize("jobs, dims, strip", [
    (48, (40, 1016), False), (48, (8, 776, 1016), False),                            # registers (shallow), 80 columns, 64
    (20, (264, 1000), False), (23, (520, 1272), False), (48, (136, 776), False),     # 96, 128, 80
    (64, (72, 640), True), (40, (136, 1024, 8), True),                               # strips: 80 columns, across their borders; 64
])
def test_evenly_spread_columns_up_to_32_rows(jobs, dims, strip):
    """Widths that end inside a tile, depths of less than a k-step and of less than the ring, 1 - 32 rows; the depth-fused launch gives
    the same bits."""
    specs = [dict(M=[1, 16, 17, 32, 7][i % 5], dims=dims, acts=([GELU, RELU] * 2)[:len(dims) - 2] + [NONE], strip=strip) for i in range(jobs)]
    outs, refs, n = run_jobs(specs, salus.BF16)
    assert n == len(dims) - 1
    fused, _, _ = run_jobs(specs, salus.BF16, fuse=True)
    for o, r, f, j in zip(outs, refs, fused, specs):
        assert np.isfinite(o).all(), j
        assert norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))
        assert np.array_equal(o.view(np.uint32), f.view(np.uint32)), j


# Tiles of up to 32 rows through LDS, one and two row tiles of each width: (jobs, widths, strips); ROWS has the rows that make
# it one row tile or two.  Depths go round the ring more than once and end inside a k-step, widths end inside a tile.
ROWS = {1: [1, 16, 7, 12, 3], 2: [1, 16, 17, 32, 7]}
SMALL_TILES = {
    "even<%d, 4>": (36, (1096, 448), False), "even<%d, 5>": (48, (1000, 776), False), "even<%d, 6>": (20, (520, 1000), False),
    "even<%d, 8>": (23, (520, 1272), False),
    "even<%d, 4>, strips": (40, (1064, 1024), True), "even<%d, 5>, strips": (30, (1064, 640), True), "even<%d, 8>, strips": (24, (2088, 1024), True),
    "even<%d, 6>, strips beside rows": (20, (520, [1024, 1000]), True), "even<%d, 8>, strips beside rows": (23, (520, [1280, 1272]), True),
    "even<%d, 4>, less than a ring": (37, (40, 800), False),
    "narrow<%d, false, 1, 0, true>": (3, (4104, 24), False), "narrow<%d, false, 2, 0, true>": (5, (1064, 1032), False),
    "narrow<%d, false, 4, 0, true>": (14, (1064, 1032), False), "narrow<%d, false, 4, 0, true>, strips": (14, (1064, 1024), True),
    "narrow<%d, false, 4, 0, true>, two launches": (100, (264, 200), False),
}
SMALL_TILES = {n.replace("%d", str(mt)): (mt, *v) for n, v in SMALL_TILES.items() for mt in (1, 2)}


def small_tiles(name):
    """The jobs of one of them and the kernels that they launch."""
    mt, jobs, (K, N), strip = SMALL_TILES[name]
    N = N if isinstance(N, list) else [N]
    return ([dict(M=ROWS[mt][i % 5], dims=(K, N[i % len(N)]), acts=[[GELU, RELU, NONE][i % 3]], strip=strip) for i in range(jobs)],
            [name.split(">")[0] + ">"] * ((jobs + 63) // 64))


@pytest.mark.parametrize("name", SMALL_TILES)
def test_small_tiles_through_lds(name):
    """Against the oracle, and bit for bit against the depth-fused launch, whose tiles sum in the same order."""
    specs, kernels = small_tiles(name)
    outs, refs, n = run_jobs(specs, salus.BF16)
    assert n == len(kernels)
    fused, _, _ = run_jobs(specs, salus.BF16, fuse=True)
    for o, r, f, j in zip(outs, refs, fused, specs):
        assert np.isfinite(o).all(), j
        assert norm_rel_err(o, r) < TOL_BF16_TIGHT, (j, norm_rel_err(o, r))
        assert np.array_equal(o.view(np.uint32), f.view(np.uint32)), j


@pytest.mark.parametrize("jobs, dims, M", [
    (1, (4, 4), 1), (2, (132, 68, 20), 17), (3, (1028, 1004, 12), 16), (1, (60, 260, 36), 128), (4, (516, 1024, 1028), 16),
])
def test_narrow_float_tiles(jobs, dims, M):
    """Widths that end inside a tile, depths of less than a k-step per wavefront; the depth-fused launch gives the same bits."""
    specs = [dict(M=max(1, M - 5 * (i % 3)), dims=dims, acts=([GELU, RELU] * 2)[:len(dims) - 2] + [NONE]) for i in range(jobs)]
    outs, refs, _ = run_jobs(specs, salus.F32)
    fused, _, _ = run_jobs(specs, salus.F32, fuse=True)
    for o, r, f, j in zip(outs, refs, fused, specs):
        assert np.isfinite(o).all() and norm_rel_err(o, r) < TOL_F32, (j, norm_rel_err(o, r))
        assert np.array_equal(o.view(np.uint32), f.view(np.uint32)), j


def test_rows_of_infinities_stay_in_their_rows_of_a_narrow_tile():
    """K ends inside a k-step: what follows a row of X and the last row of W does not reach the sums."""
    M, K, N = 3, 40, 24
    w_offs, P, x_off, y_off, h_off, E = mlp_layout((K, N), 2, M)
    dp = DevicePool(P + 4096 + E, policy=salus.POLICY_PACK)
    rng = np.random.default_rng(3)
    W = synth.f32_to_bf16_bits((rng.standard_normal((K, N)) / np.sqrt(K)).astype(np.float32))
    X = synth.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    ref = dense.mlp_forward_bf16(X, [W], [NONE])[-1]
    X[1] = 0x7f80
    st, job = dp.pool.lane_alloc(P + 4096, E, 0, 1)
    assert st == salus.OK
    q = dp.pool.job_query(job)
    dp.write(q.persist_off, W)
    dp.write(q.persist_off + W.nbytes, np.full(4096 // 2, 0x7fc0, np.uint16))      # NaN right behind the weights
    dp.write(q.lane_off + x_off, X)
    descs, keep = salus.Pool.make_descs([dict(job=job, M=M, dtype=salus.BF16, layers=[(K, N, 0, NONE)], x_off=x_off, y_off=y_off, h_off=h_off)])
    assert dp.pool.grouped_forward(descs, stream=dp.stream) == salus.OK
    dp.sync()
    Y = dp.read(q.lane_off + y_off, M * N * 4, np.float32).reshape(M, N)
    assert not np.isfinite(Y[1]).any()
    assert norm_rel_err(Y[[0, 2]], ref[[0, 2]]) < TOL_BF16_TIGHT
    dp.close()
