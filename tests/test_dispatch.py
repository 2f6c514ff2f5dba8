"""Which kernels the library launches for a round (CPU only: launch_recorder.c stands in for the HIP runtime, so the launch
code itself runs and nothing else does)."""
import json
import os
import re
import subprocess
import sys

import pytest

from paper_1902_04610_amd import build

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
    K, N = max(case["K"]), case["N"]
    up = lambda v: (v + 255) // 256 * 256
    top = max(case["rows"])
    P, y = up(K * N * esz), up(top * K * esz)
    E = y + up(top * N * 4)
    p = pool(len(case["rows"]) * (P + E))
    items = []
    for M, k in zip(case["rows"], case["K"]):
        st, job = p.lane_alloc(P, E, 0, 1)
        assert st == salus.OK
        items.append(dict(job=job, M=M, dtype=dt, layers=[(k, N, 0, salus.ACT_NONE)], x_off=0, y_off=y, h_off=E))
    descs, keep = salus.Pool.make_descs(items)
    take()
    assert p.grouped_forward(descs, stream=STREAM) == salus.OK, p.last_error()
    out = take().decode()
    p.close()
    return out

CASES = json.load(sys.stdin)
print(json.dumps([globals()[c["do"]](c) for c in CASES]))
""" % STREAM


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    """Runs cases in a child process; a list of lines for each, kernel names demangled and without arguments."""
    if not os.path.exists(build.LIB):
        build.build()
    so = str(tmp_path_factory.mktemp("recorder") / "librecorder.so")
    subprocess.check_call(["gcc", "-O1", "-fPIC", "-shared", "-Wall", "-o", so, os.path.join(HERE, "launch_recorder.c")])

    def run(cases):
        env = dict(os.environ, LD_PRELOAD=":".join(filter(None, [so, os.environ.get("LD_PRELOAD")])), PYTHONPATH=build.ROOT)
        r = subprocess.run([sys.executable, "-c", CHILD], input=json.dumps(cases), cwd=build.ROOT, env=env, stdout=subprocess.PIPE,
                           stderr=subprocess.PIPE, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        logs = json.loads(r.stdout.splitlines()[-1])
        plain = subprocess.run(["c++filt"], input="----\n".join(logs), stdout=subprocess.PIPE, text=True, check=True).stdout
        return [re.sub(r"(?:void )?salus::|\(.*?\)", "", p).split("\n") for p in plain.split("----\n")]

    return run


def kernels(lines):
    return [line.rsplit(" ", 3)[0][len("launch "):] for line in lines if line.startswith("launch ")]


def case(rows, K, N, dtype="bf16"):
    """Jobs of one layer; K one for all or one for each."""
    return dict(do="forward", rows=rows, K=K if isinstance(K, list) else [K] * len(rows), N=N, dtype=dtype)


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
        case([256, 333], [64, 264], 72),                                   # few, but beside a job that takes it anyway
    ]
    for c, log in zip(many, record(many)):
        assert len(kernels(log)) == 1 and kernels(log)[0].startswith("grouped_dense_bf16_tiled<"), (c, kernels(log))


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
        ([32] * 4, 1204, 780, 1), ([64] * 8, 512, 512, 1), ([16] * 40, 516, 1204, 1), ([8] * 8 + [32] * 4, 1536, 1536, 1),
        ([128] * 12, 1536, 1536, 2), ([40] * 12, 1536, 1536, 2), ([33, 80] * 20, 1536, 1536, 2), ([40] * 40, 1024, 1024, 2),
        ([40] * 20, 1536, 1536, 4), ([64] * 40, 1536, 1536, 4), ([128] * 40, 1024, 1024, 4), ([33] * 30, 1024, 1024, 4),     # whole rounds
        ([200] * 12, 516, 1204, 4),
    )])
