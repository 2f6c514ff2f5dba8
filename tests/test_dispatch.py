"""Which kernels the library launches for a round (CPU only: launch_recorder.c stands in for the HIP runtime, so the launch
code itself runs and nothing else does)."""
import json
import os
import re
import subprocess
import sys

import pytest

from paper_1902_04610_amd import build
from test_gpu_routes import SMALL_TILES, small_tiles

HERE = os.path.dirname(os.path.abspath(__file__))
STREAM = 0x50                        # any handle

CHILD = r"""
import ctypes, json, sys
from paper_1902_04610_amd import salus
take = ctypes.CDLL(None).recorder_take
take.restype = ctypes.c_char_p
BASE, STREAM = 1 << 40, %d

def pool(capacity, **kw):
    return salus.Pool(BASE, capacity, stream=STREAM, policy=salus.POLICY_PACK, **kw)

def forward(case):
    dt = salus.F32 if case["dtype"] == "f32" else salus.BF16
    esz = 4 if dt == salus.F32 else 2
    up = lambda v: (v + 255) // 256 * 256
    top, layers = max(case["rows"]), []
    for dims, strip in zip(case["dims"], case["strip"]):
        at, mine = 0, []
        for k, n in zip(dims, dims[1:]):
            mine.append((k, n, at, salus.ACT_NONE, salus.LAYOUT_STRIP128 if strip and n %% 128 == 0 else salus.LAYOUT_ROWMAJOR))
            at += up(k * n * esz)
        layers.append((at, mine))
    P, y = max(size for size, _ in layers), up(top * max(dims[0] for dims in case["dims"]) * esz)
    h = y + up(top * max(dims[-1] for dims in case["dims"]) * 4)
    E = h + max(salus.forward_work_bytes(top, [t[:4] for t in mine], dt) for _, mine in layers)
    p = pool(len(case["rows"]) * (P + E) + sum(v + 256 for v in case["idle"]))
    for v in case["idle"]:
        st, other = p.lane_alloc(v, 256, 0, 0)
        assert st == salus.OK
    items = []
    for M, (_, mine) in zip(case["rows"], layers):
        st, job = p.lane_alloc(P, E, 0, 1)
        assert st == salus.OK
        items.append(dict(job=job, M=M, dtype=dt, layers=mine, x_off=0, y_off=y, h_off=h))
    if case["evicted"]:
        assert p.switch_out(other) == salus.OK
    descs, keep = salus.Pool.make_descs(items)
    take()
    assert p.grouped_forward(descs, stream=STREAM) == salus.OK, p.last_error()
    out = take().decode()
    p.close()
    return out

def train(case):
    up = lambda v: (v + 255) // 256 * 256
    jobs = []
    for M, dims in zip(case["rows"], case["dims"]):
        layers, at = [], 0
        for k, n in zip(dims, dims[1:]):
            layers.append((k, n, at, at + up(k * n * 2)))
            at += up(k * n * 2) + up(k * n * 4)
        lab = up(M * dims[0] * 2)
        logits = lab + up(M * 4)
        loss = logits + up(M * dims[-1] * 4)
        jobs.append((M, layers, at, lab, logits, loss, loss + 256 + salus.train_work_bytes(M, layers)))
    p = pool(sum(j[2] + j[6] for j in jobs) + sum(v + 256 for v in case["idle"]) + 4096)
    for v in case["idle"]:
        assert p.lane_alloc(v, 256, 0, 0)[0] == salus.OK
    items = []
    for M, layers, P, lab, logits, loss, E in jobs:
        st, job = p.lane_alloc(P, E, 0, 1)
        assert st == salus.OK
        items.append(dict(job=job, M=M, lr=0.1, layers=layers, x_off=0, labels_off=lab, logits_off=logits, loss_off=loss, work_off=loss + 256))
    descs, keep = salus.Pool.make_train_descs(items)
    take()
    assert p.grouped_train_step(descs, stream=STREAM) == salus.OK, p.last_error()
    out = take().decode()
    p.close()
    return out

def compaction(case):
    # two blocks above a hole smaller than either: one in-place move; then the same again above the next hole
    p = pool(1 << 30, max_lanes=1)
    created = take().decode()
    for size in (1 << 20, 8 << 20, 2 << 20, 16 << 20):
        assert p.lane_alloc(size, 4096, 0, 0)[0] == salus.OK
    out = [created]
    for job in (0, 2):
        assert p.lane_free(job) >= 0
        take()
        assert len(p.compact()) >= 1
        out.append(take().decode())
    p.close()
    return "====\n".join(out)

class SlideState(ctypes.Structure):
    _fields_ = [("progress", ctypes.c_void_p), ("epoch", ctypes.c_uint32), ("failed", ctypes.c_void_p), ("failed_dev", ctypes.c_void_p),
                ("max_grid", ctypes.c_uint32), ("spin_limit", ctypes.c_uint32)]

def slides(case):
    lib = salus.lib()
    state = SlideState()
    assert lib._ZN5salus18slide_state_createEPNS_10SlideStateE(ctypes.byref(state)) == 0
    one = lambda v: ctypes.byref(ctypes.c_uint64(v))
    take()
    out = []
    for epoch in case["epochs"]:
        if epoch is not None:
            state.epoch = epoch
        assert lib._ZN5salus12launch_slideEPcPKmS2_S2_jPNS_10SlideStateEP12ihipStream_tPm(
            ctypes.c_void_p(BASE), one(4096), one(0), one(300 << 20), 1, ctypes.byref(state), ctypes.c_void_p(STREAM), None) == 0
        out.append("%%d\n" %% state.epoch + take().decode())
    return "====\n".join(out)

CASES = json.load(sys.stdin)
print(json.dumps([globals()[c["do"]](c) for c in CASES]))
""" % STREAM


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    """Runs cases in a child process; a list of lines for each, kernel names demangled and, unless asked for, without arguments."""
    if not os.path.exists(build.LIB):
        build.build()
    so = str(tmp_path_factory.mktemp("recorder") / "librecorder.so")
    subprocess.check_call(["gcc", "-O1", "-fPIC", "-shared", "-Wall", "-o", so, os.path.join(HERE, "launch_recorder.c")])

    def run(cases, arguments=False):
        env = dict(os.environ, LD_PRELOAD=":".join(filter(None, [so, os.environ.get("LD_PRELOAD")])), PYTHONPATH=build.ROOT)
        r = subprocess.run([sys.executable, "-c", CHILD], input=json.dumps(cases), cwd=build.ROOT, env=env, stdout=subprocess.PIPE,
                           stderr=subprocess.PIPE, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        logs = json.loads(r.stdout.splitlines()[-1])
        plain = subprocess.run(["c++filt"], input="----\n".join(logs), stdout=subprocess.PIPE, text=True, check=True).stdout
        return [re.sub(r"(?:void )?salus::" + ("" if arguments else r"|\(.*?\)"), "", p).split("\n") for p in plain.split("----\n")]

    return run


def kernels(lines):
    return [line.rsplit(" ", 3)[0][len("launch "):] for line in lines if line.startswith("launch ")]


def case(rows, K, N, dtype="bf16", strip=False, idle=(), evicted=False):
    """Jobs of one layer, or of as many as N has widths; K and strip one for all or one for each.  idle: bytes of jobs that the
    pool holds besides; evicted: the last of them has been switched out."""
    each = lambda v: v if isinstance(v, list) else [v] * len(rows)
    dims = [[k] + (N if isinstance(N, list) else [N]) for k in each(K)]
    return dict(do="forward", rows=rows, dims=dims, dtype=dtype, strip=each(strip), idle=list(idle), evicted=evicted)


def check(record, expected):
    """(case, kernels) pairs"""
    for (c, want), log in zip(expected, record([c for c, _ in expected])):
        assert kernels(log) == want, (c, kernels(log))


def test_ragged_depth_few_tiles(record):
    """More than 128 rows, K no multiple of 64, too few tiles to fill the chip: one launch of register tiles for all jobs."""
    check(record, [(c, ["grouped_dense_bf16<2, false, false>"]) for c in (
        case([256], 3080, 776), case([192] * 4, 1032, 72), case([600], 200, 264), case([130] * 10, 776, 1016),
        case([129, 150, 191, 192, 250, 300, 400], 1000, 384),        # rows on either side of 192
    )])


def test_ragged_depth_many_tiles(record):
    """With enough of them, or beside jobs of other shapes: one launch of the tiled kernel, whatever the rows."""
    many = [
        case([150, 191, 192, 260] * 5, 1000, 1016), case([129] * 30, 200, 1000), case([200] * 10, 3080, 776),
        case([256, 333], [320, 264], 72),                                   # few, but beside a job that takes it anyway
    ]
    for c, log in zip(many, record(many)):
        assert len(kernels(log)) == 1 and kernels(log)[0].startswith("grouped_dense_bf16_tiled<"), (c, kernels(log))


def test_shallow_layers_above_128_rows(record):
    """K of up to 256, a multiple of 64: the same rule; 128 rows take the kernels of smaller jobs when there are few."""
    check(record, [(case(rows, K, N), ["grouped_dense_bf16" + kernel]) for rows, K, N, kernel in (
        ([256], 64, 4096, "<2, false, false>"), ([160] * 8, 128, 1024, "<2, false, false>"), ([700], 256, 2048, "<2, false, false>"),
        ([128], 64, 1024, "_narrow<2, false, 2, 8, false>"), ([128] * 8, 256, 1024, "_stream<64, 64, 2, 1, 2, false, 4>"),
        ([128] * 32, 64, 1024, "_tiled<128, 128, 2, 2>"), ([300] * 8, 256, 4096, "_tiled<128, 128, 2, 2>"),
        ([256], 320, 4096, "_tiled<128, 128, 2, 2>"),
    )])


def test_rows_33_to_128(record):
    """Narrow register tiles while there is at most one per compute unit, the ring or (deep, full) 64-row tiles beyond."""
    check(record, [(case(rows, K, N), ["grouped_dense_bf16_" + kernel]) for rows, K, N, kernel in (
        ([33], 1024, 64, "narrow<2, false, 2, 8, false>"), ([48] * 4, 64, 1024, "narrow<2, false, 2, 8, false>"),       # 32-column tiles
        ([33, 127, 64], 4096, 1032, "narrow<2, false, 4, 4, false>"), ([33] * 16, 128, 512, "narrow<2, false, 4, 4, false>"),     # 64-column tiles
        ([33] * 24, 1024, 512, "stream<64, 64, 2, 1, 2, false, 4>"), ([33] * 17, 128, 512, "stream<64, 64, 2, 1, 2, false, 4>"),
        ([64] * 40, 520, 1032, "stream<64, 128, 2, 2, 1, false, 3>"), ([48] * 64, 1024, 4096, "rows64"),
    )])


def test_float_row_tiles(record):
    check(record, [(case(rows, K, N, "f32"), ["grouped_dense_f32<%d>" % tile]) for rows, K, N, tile in (
        ([32] * 12, 1204, 780, 2), ([17] * 30, 1536, 384, 2),       # 312 and 360 16-row tiles: 32-row ones, each on a compute unit of its own
        ([32] * 4, 1204, 780, 1), ([32] * 40, 256, 256, 1), ([64] * 8, 512, 512, 1), ([16] * 40, 516, 1204, 1), ([8] * 8 + [32] * 4, 1536, 1536, 1),
        ([128] * 12, 1536, 1536, 2), ([40] * 12, 1536, 1536, 2), ([33, 80] * 20, 1536, 1536, 2), ([40] * 40, 1024, 1024, 2),
        ([40] * 20, 1536, 1536, 4), ([64] * 40, 1536, 1536, 4), ([128] * 40, 1024, 1024, 4), ([33] * 30, 1024, 1024, 4),     # whole rounds
        ([200] * 12, 516, 1204, 4),
    )])


def test_a_compaction_allocates_nothing_and_waits_for_its_own_stream(record):
    """The first in-place move of a pool like every other: what it needs was there when the pool was created."""
    (log,) = record([dict(do="compaction")])
    created, first, second = "\n".join(log).split("====\n")
    assert "hipMalloc" in created
    for lines in (first, second):
        assert re.findall(r"^hip(?:Host)?(?:Malloc|Free).*", lines, re.M) == []
        assert set(re.findall(r"^hip(?:Stream|Device)Synchronize.*", lines, re.M)) == {"hipStreamSynchronize %#x" % STREAM}
    # counters are cleared by a launch on that stream, once
    assert re.findall(r"launch (slide_\w+)", first) == ["slide_clear", "slide_down"]
    assert re.findall(r"launch (slide_\w+)", second) == ["slide_down"]


def test_counters_of_the_in_place_move_never_wrap(record):
    """A workgroup's counter may rest for any number of launches; the difference to the epoch is taken in 32 bits with a sign."""
    (log,) = record([dict(do="slides", epochs=[None, None, (1 << 30) - 1, None, None, (1 << 31) - 2, None])])
    runs = [r.split("\n", 1) for r in "\n".join(log).split("====\n")]
    assert all(0 < int(epoch) <= (1 << 30) + 16 for epoch, _ in runs)
    assert [re.findall(r"launch (slide_\w+)", lines) for _, lines in runs] == \
        [["slide_clear", "slide_down"], ["slide_down"], ["slide_down"], ["slide_clear", "slide_down"], ["slide_down"],
         ["slide_clear", "slide_down"], ["slide_down"]]


def test_two_tiles_of_128_by_256_per_compute_unit(record):
    """Where they leave less of the last round empty than 256 x 256 or waste less of it than 128 x 128; 256 of them only if the
    launch is bound by weights (up to 128 rows)."""
    check(record, [(case(rows, K, N), ["grouped_dense_bf16_tiled" + kernel]) for rows, K, N, kernel in (
        ([65] * 64, 320, 1024, "<128, 256, 1, 4>"), ([100] * 64, 1024, 1024, "<128, 256, 1, 4>"),
        ([293, 300, 299] * 11, [320, 320, 328] * 11, 1544, "<128, 256, 1, 4>"), ([100] * 64, 384, 1544, "<128, 256, 1, 4>"),
        ([100] * 48, 1024, 1024, "<128, 256, 2, 4>"), ([200] * 24, 1024, 1024, "<128, 256, 2, 4>"),
        ([500] * 4, 2048, 2048, "<128, 128, 2, 2>"), ([4096] * 4, 1024, 4096, "<256, 256, 2, 4>"),
    )])


def test_narrow_tiles_up_to_32_rows(record):
    """The fewest columns that leave at most one tile per compute unit, 16 at least; 128 once 64 leave more."""
    check(record, [(case(rows, K, N), ["grouped_dense_bf16" + kernel]) for rows, K, N, kernel in (
        ([1], 4096, 4096, "_narrow<1, false, 1, 0, true>"), ([17] * 4, 1024, 1024, "_narrow<2, false, 1, 0, true>"),
        ([16] * 5, 1024, 1024, "_narrow<1, false, 2, 0, true>"), ([17] * 8, 1024, 1024, "_narrow<2, false, 2, 0, true>"),
        ([32] * 9, 1024, 1024, "_narrow<2, false, 4, 0, true>"), ([8] * 16, 1024, 1024, "_narrow<1, false, 4, 0, true>"),
        ([8] * 17, 1024, 1024, "<1, false, true>"), ([1], 8, 1 << 22, "<1, false, true>"),
    )])


def test_columns_spread_evenly_up_to_32_rows(record):
    """Tiles of 64 - 128 columns where 128 load compute units unevenly; registers where they do not, and for whole lines from HBM."""
    even = "_even<%d, %d>"
    check(record, [(case(rows, K, N), ["grouped_dense_bf16" + kernel]) for rows, K, N, kernel in (
        ([8] * 48, 512, 1016, even % (1, 4)), ([17] * 48, 1000, 776, even % (2, 5)), ([8] * 20, 264, 1000, even % (1, 6)),
        ([8] * 23, 520, 1272, even % (1, 8)), ([32] * 20, 1032, 2048, even % (2, 4)), ([8] * 64, 128, 640, even % (1, 5)),
        ([8] * 64, 4096, 1024, "<1, false, true>"), ([32] * 64, 1000, 3080, "<2, false, true>"), ([8] * 24, 8000, 1160, "<1, false, true>"),
        ([8] * 40, 4096, 1024, "<1, false, true>"),
    )])


def test_narrow_float_tiles(record):
    """16 columns while that is at most one tile per compute unit."""
    check(record, [(case(rows, K, N, "f32"), ["grouped_dense_f32" + kernel]) for rows, K, N, kernel in (
        ([1], 4, 4, "_narrow"), ([16] * 4, 1024, 1024, "_narrow"), ([16] * 4, 1024, 1028, "<1>"), ([128], 60, 512, "_narrow"), ([129], 60, 512, "<1>"),
    )])


def test_columns_spread_evenly_while_all_that_is_resident_fits_the_cache(record):
    """What decides is what the pool's jobs hold, not what this round reads; several layers, strips."""
    even = "grouped_dense_bf16_even<1, %d>"
    registers = "grouped_dense_bf16<1, false, true>"
    small = ([8] * 30, 2048, 640)
    check(record, [
        (case(*small), [even % 5]), (case(*small, idle=[200 << 20]), [registers]),
        (case(*small, idle=[200 << 20], evicted=True), [even % 5]), (case(*small, idle=[100 << 20, 100 << 20], evicted=True), [even % 5]),
        # 3 layers of together 8.5 MB a job, every one of which would fit by itself
        (case([8] * 28, 2048, [640, 2304, 640]), [registers] * 3), (case([8] * 27, 2048, [640, 2304, 640]), [even % 5, registers, even % 5]),
        (case([8] * 30, 2048, 640, strip=True), [even % 5]), (case([8] * 30, 2048, 640, strip=True, idle=[200 << 20]), [registers]),
        (case([8] * 36, 2048, 448), [even % 4]), (case([8] * 36, 2048, 448, idle=[200 << 20]), [even % 4]),       # almost half the load
        # from further away: only rows that begin inside a line, and only where the load falls by a tenth
        (case([8] * 48, 6160, 776), [even % 5]), (case([8] * 48, 1000, 776, idle=[400 << 20]), [even % 5]),
        (case([8] * 23, 520, 1272), [even % 8]), (case([8] * 23, 520, 1272, idle=[400 << 20]), [registers]),
    ])


def test_whole_lines_one_tile_per_compute_unit(record):
    """128 columns through LDS only for jobs of 17 rows and more, in layers deeper than 2048 (up to 192 tiles) or 3072; narrower ones that are
    still one per compute unit from 1024; never 96."""
    check(record, [(case(rows, K, N), ["grouped_dense_bf16" + kernel]) for rows, K, N, kernel in (
        ([8] * 47, 1152, 512, "<1, false, true>"), ([2] * 9, 1536, 2688, "<1, false, true>"), ([16] * 23, 2048, 1024, "<1, false, true>"),
        ([16] * 23, 2056, 1024, "_even<1, 8>"), ([17] + [8] * 19, 1664, 1408, "_even<2, 8>"), ([8] * 30, 1032, 640, "_even<1, 5>"),
        ([8] * 30, 1024, 640, "<1, false, true>"), ([8] * 24, 2056, 1024, "_even<1, 8>"), ([8] * 25, 3072, 1024, "<1, false, true>"),
        ([8] * 25, 3080, 1024, "_even<1, 8>"),
    )])


def test_rows_inside_lines_in_shallow_layers(record):
    """From the cache LDS tiles always, in layers below 320 only where the load falls by a fifth; from further away where it falls by
    a tenth, in layers below 512 by three tenths."""
    far = dict(idle=[400 << 20])
    check(record, [(case(rows, K, N, **kw), ["grouped_dense_bf16" + kernel]) for rows, K, N, kw, kernel in (
        ([8] * 64, 256, 424, {}, "<1, false, true>"), ([1] * 64, 184, 1560, {}, "<1, false, true>"), ([8] * 30, 224, 1464, {}, "_even<1, 6>"),
        ([8] * 64, 312, 424, {}, "<1, false, true>"), ([8] * 64, 320, 424, {}, "_even<1, 8>"), ([32] * 64, 680, 1752, {}, "_even<2, 8>"),
        ([8] * 21, 424, 3752, far, "<1, false, true>"), ([8] * 64, 448, 696, far, "<1, false, true>"), ([8] * 10, 384, 3304, far, "_even<1, 5>"),
        ([8] * 64, 512, 696, far, "_even<1, 6>"), ([8] * 64, 520, 424, far, "<1, false, true>"),
    )])


def test_more_jobs_than_a_launch_holds(record):
    """Every launch of 64 jobs takes the tiles that suit it, whatever the others hold."""
    check(record, [
        (case([8] * 100, 1024, 200), ["grouped_dense_bf16_narrow<1, false, 4, 0, true>"] * 2),
        (case([8] * 65, 512, 1016), ["grouped_dense_bf16_even<1, 8>", "grouped_dense_bf16_narrow<1, false, 1, 0, true>"]),
        (case([8] * 64 + [17] * 17, 1032, 1024), ["grouped_dense_bf16<1, false, true>", "grouped_dense_bf16_even<2, 5>"]),
        (case([8] * 128, 512, 64, "f32"), ["grouped_dense_f32_narrow"] * 2),
        (case([8] * 65, 512, 256, "f32"), ["grouped_dense_f32<1>", "grouped_dense_f32_narrow"]),
    ])


def test_one_round_of_256_by_256_from_further_away_than_the_cache(record):
    """It is not traded for a round and a bit of 128 x 128 tiles there; launches of several rounds choose alike."""
    far = dict(idle=[400 << 20])
    check(record, [(case(rows, K, N, **kw), ["grouped_dense_bf16_tiled" + kernel]) for rows, K, N, kw, kernel in (
        ([500] * 5, 1280, 3968, {}, "<128, 128, 2, 2>"), ([500] * 5, 1280, 3968, far, "<256, 256, 2, 4>"),
        ([500] * 5, 1280, 3968, dict(idle=[400 << 20], evicted=True), "<128, 128, 2, 2>"),
        ([1000] * 29, 512, 768, {}, "<128, 256, 1, 4>"), ([1000] * 29, 512, 768, far, "<128, 256, 1, 4>"),
    )])


def test_parity_tests_of_small_tiles_launch_what_they_are_named_after(record):
    cases = [small_tiles(name) for name in SMALL_TILES]
    check(record, [(dict(do="forward", rows=[j["M"] for j in specs], dims=[j["dims"] for j in specs], dtype="bf16",
                         strip=[j["strip"] for j in specs], idle=[], evicted=False), ["grouped_dense_bf16_" + k for k in names])
                   for specs, names in cases])


def test_weights_of_up_to_128_rows_from_further_away_are_asked_for_once(record):
    far, once, plain = dict(idle=[240 << 20]), "_once<128, 256, 1, 4>", "<128, 256, 1, 4>"
    check(record, [(case(rows, K, N, **kw), ["grouped_dense_bf16_tiled" + kernel]) for rows, K, N, kw, kernel in (
        ([100] * 64, 1024, 1024, {}, plain), ([100] * 64, 1024, 1024, far, once), ([128] * 64, 1024, 1024, far, once),
        ([1000] * 29, 512, 768, far, plain),
    )])
    from test_gpu_once_and_few import ONCE
    check(record, [(dict(case([M] * min(jobs, 64), K, N, strip=strip, **far)), ["grouped_dense_bf16_tiled" + once]) for jobs, M, K, N, strip in ONCE])


def test_half_line_cases_take_64_by_64_tiles(record):
    """The first layers of the GPU test of bf16 results in half lines."""
    for jobs, K, N, M in ((24, 136, 520, 33), (20, 72, 536, 64), (12, 264, 1000, 65), (7, 200, 1064, 127)):
        check(record, [(case([max(33, M - 5 * (i % 4)) for i in range(jobs)], K, N), ["grouped_dense_bf16_stream<64, 64, 2, 1, 2, false, 4>"])])


def test_jobs_of_128_rows_and_more_that_are_few(record):
    """The smallest tile of which there is at most one per compute unit; 64 x 128, two per compute unit, where 128 x 128 tiles are more
    than one; shallower layers, rounds with smaller jobs and more tiles as before."""
    from test_gpu_few_tiles import FEW
    check(record, [(case(rows, K, N, strip=strip), ["grouped_dense_bf16_" + kernel]) for rows, K, N, strip, kernel in FEW + [
        ([256], 320, 4096, False, "tiled<128, 128, 2, 2>"), ([500] * 4, 2048, 2048, False, "tiled<128, 128, 2, 2>"),
        ([200] * 24, 1024, 1024, False, "tiled<128, 256, 2, 4>"), ([128] * 33, 384, 1024, False, "tiled<128, 128, 2, 2>"),
    ]])


def test_float_32_row_tiles_one_per_compute_unit(record):
    """Layers deeper than 256 with more than one 16-row tile and at most one 32-row tile per compute unit."""
    mixed = [1, 1, 2, 3, 4, 8, 9, 12, 14, 31, 76, 77]
    check(record, [(case(rows, K, N, "f32"), ["grouped_dense_f32<%d>" % tile]) for rows, K, N, tile in (
        (mixed, 1204, 780, 2), (mixed, 516, 1204, 1), (mixed, 780, 388, 1), ([86] * 5, 1012, 936, 2), ([125] * 2, 1484, 1136, 2),
        ([95] * 5, 260, 696, 2), ([95] * 5, 256, 696, 1), ([68] * 8, 988, 760, 1), ([16] * 40, 516, 452, 1),
    )])


def test_half_a_round_of_128_by_256_from_further_away(record):
    """Where two tiles per compute unit would leave most of them idle, weights from further away change nothing."""
    for kw in ({}, dict(idle=[240 << 20])):
        check(record, [(case([33, 67] * 5, 1792, 3456, strip=True, **kw), ["grouped_dense_bf16_tiled<128, 256, 2, 4>"])])


def test_float_row_tiles_of_every_launch(record):
    """One 32-row tile per compute unit is a matter of the launch, not of all jobs of the round."""
    check(record, [(case([M] * jobs, K, N, "f32"), ["grouped_dense_f32" + k for k in names]) for jobs, M, K, N, names in (
        (90, 48, 900, 64, ["<1>", "<1>"]), (65, 60, 1204, 68, ["<2>", "_narrow"]), (128, 48, 388, 128, ["<2>", "<2>"]), (64, 48, 900, 64, ["<1>"]),
    )])


def test_float_layers_with_four_steps_in_flight(record):
    """16-row tiles of layers 257 - 320, 449 - 512 and 768 more deep, from further away 193 - 256 too, in every launch for itself."""
    far = [240 << 20]
    expected = [(12, 16, 256, 1204, [], 0), (12, 16, 260, 1204, [], 1), (12, 16, 320, 1204, [], 1), (12, 16, 324, 1204, [], 0), (12, 16, 448, 1204, [], 0),
                (12, 16, 452, 1204, [], 1), (12, 16, 512, 1204, [], 1), (12, 16, 516, 1204, [], 0), (12, 16, 192, 1204, far, 0), (12, 16, 196, 1204, far, 1),
                (12, 16, 256, 1204, far, 1), (12, 16, 196, 1204, [], 0), (12, 16, 384, 1204, far, 0), (82, 2, 276, 944, [], 2), (5, 16, 276, 1500, [], 1),
                (12, 30, 276, 780, [], 0), (12, 16, 1024, 1204, [], 0), (12, 16, 1028, 1204, [], 1), (12, 16, 1280, 1204, [], 1), (12, 16, 1284, 1204, far, 0)]
    logs = record([case([M] * jobs, K, N, "f32", idle=idle) for jobs, M, K, N, idle, _ in expected], arguments=True)
    for (jobs, M, K, N, idle, count), log in zip(expected, logs):
        found = kernels(log)
        assert sum("FourInFlight" in k for k in found) == count and len(found) == max(count, 1), (jobs, M, K, N, found)


def test_whole_lines_from_further_away_take_the_tiles_that_the_cache_gives(record):
    """128 x 256 tiles that ask for weights once are preferred beyond their time only where rows of an operand begin inside a line."""
    far = dict(idle=[400 << 20])
    check(record, [(case([M] * jobs, K, N, strip=strip, **far), ["grouped_dense_bf16_tiled" + kernel]) for jobs, M, K, N, strip, kernel in (
        (55, 110, 1024, 1280, True, "<128, 128, 2, 2>"), (23, 100, 768, 3072, False, "<128, 128, 2, 2>"), (26, 100, 1536, 2688, True, "<128, 128, 2, 2>"),
        (63, 90, 1616, 1168, False, "_once<128, 256, 1, 4>"), (46, 80, 2344, 3072, False, "_once<128, 256, 1, 4>"),
        (56, 110, 2048, 1528, False, "_once<128, 256, 1, 4>"),
    )])


def training(rows, dims, far=False):
    """One training step; rows and dims of every job, dims one for all or one for each."""
    return dict(do="train", rows=rows, dims=[list(d) for d in (dims if isinstance(dims, list) else [dims] * len(rows))], idle=[240 << 20] if far else [])


def test_parity_tests_of_tails_and_of_the_ring_launch_what_they_are_named_after(record):
    from test_gpu_tiles import RING_GRADIENTS, TAILS
    check(record, [(case([M - i % 3 for i in range(jobs)], K, N, strip=strip), ["grouped_dense_bf16_tiled<128, 128, 2, 2>"]) for jobs, M, K, N, strip in TAILS])
    for (jobs, dims, M, columns), log in zip(RING_GRADIENTS, record([training([M] * jobs, dims) for jobs, dims, M, _ in RING_GRADIENTS])):
        assert kernels(log)[3:-1] == ["grouped_dense_bf16_stream<64, 64, 2, 1, 2, true, 4>" if columns == 64 else
                                      "grouped_dense_bf16_stream<64, 128, 2, 2, 1, true, 3>"], (dims, M, kernels(log))


def test_input_gradients_in_narrow_tiles(record):
    """32 x 32 register tiles of at most one per compute unit (256 and 260 of them)."""
    for (rows, dims, kernel), log in zip(*(lambda cs: (cs, record([training(r, d) for r, d, _ in cs])))([
        ([127], (72, 2048, 264), "narrow<2, true, 2, 8, false>"), ([127], (72, 2056, 264), "stream<64, 64, 2, 1, 2, true, 4>"),
        ([128] * 4, (40, 512, 72), "narrow<2, true, 2, 8, false>"), ([128] * 4, (40, 520, 72), "stream<64, 64, 2, 1, 2, true, 4>"),
    ])):
        assert kernels(log)[3:-1] == ["grouped_dense_bf16_" + kernel], (rows, dims, kernels(log))


def test_updates(record):
    """Blocks of 32 x 64 up to a mean of 88 rows (128 from further away) where more of 64 x 64 are there than run at once, LDS tiles from 192."""
    from test_gpu_updates import DIMS, MANY
    few, tall, lds = ("grouped_dw_sgd" + k for k in ("_few_rows", "", "_tiled"))
    expected = [([m] * MANY, DIMS, far, kernel) for m, far, kernel in (
        (1, False, few), (88, False, few), (89, False, tall), (191, False, tall), (192, False, lds), (89, True, few), (128, True, few), (129, True, tall))]
    expected += [([100, 150] * 6, DIMS, True, few), ([100, 158] * 6, DIMS, True, tall), ([8] * 11 + [900], DIMS, False, few),
                 ([64] * 6, DIMS, False, tall), ([64] * 7, DIMS, False, few),          # 474 and 553 blocks of 64 x 64
                 ([64] * 4, (1024, 2048), False, tall), ([64] * 4, (1032, 2048), False, few)]      # 512 and 544
    for (rows, dims, far, kernel), log in zip(expected, record([training(r, d, f) for r, d, f, _ in expected])):
        assert kernels(log)[-1] == kernel, (rows, dims, far, kernels(log))


def test_mean_losses(record):
    """In the update's launch where every job has a place for its row losses, else by a launch of their own."""
    expected = [([64], [(40, 64, 64)], True), ([65], [(40, 64)], True), ([17], [(40, 72)], False), ([17], [(72, 72, 72)], False), ([16], [(40, 64, 64)], False),
                ([64, 16, 17], [(40, 64, 72), (72, 40), (40, 8)], False), ([64, 40], [(40, 64, 64), (40, 64, 72)], True)]
    for (rows, dims, own), log in zip(expected, record([training(r, d) for r, d, _ in expected])):
        assert kernels(log).count("loss_mean") == int(own), (rows, dims, kernels(log))


def test_arguments_of_eight_and_nine_problems(record):
    """The kernels of the GPU test, and the shorter arguments up to eight problems where a kernel has them."""
    from test_gpu_few_problems import EDGE
    for jobs in (8, 9):
        cases = [case([M - (i % 3 if M > 3 else 0) for i in range(jobs)], dims[0], list(dims[1:]), dtype) for dtype, M, dims, _ in EDGE]
        for (dtype, M, dims, names), log in zip(EDGE, record(cases, arguments=True)):
            found = kernels(log)
            assert [k.split("(")[0] for k in found] == ["grouped_dense_" + k for k in names], (jobs, dtype, M, dims, found)
            for k in found:
                assert ("FewArgs" in k) == (jobs == 8 and "stream" not in k), (jobs, k)
