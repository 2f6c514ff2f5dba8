"""What the compiler makes of the device code (CPU only: every kernel file is compiled for gfx950, nothing is run)."""
import concurrent.futures
import os
import re
import subprocess

import pytest

from paper_1902_04610_amd import build

FILES = [s for s in build.SOURCES if s.startswith("kernels_")]


def compile_device(source, out, *flags):
    """Device half of one file with the library's flags; returns the compiler's remarks."""
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-O3", "-std=c++17",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(build.ROOT, "include"),
                        "-I", build.CSRC, "--cuda-device-only", "-S", *flags, "-o", str(out), os.path.join(build.CSRC, source)],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return r.stdout


@pytest.fixture(scope="module")
def ir(tmp_path_factory):
    """LLVM IR of each kernel file, as lines."""
    d = tmp_path_factory.mktemp("ir")
    with concurrent.futures.ThreadPoolExecutor(4) as pool:
        list(pool.map(lambda f: compile_device(f, d / f, "-emit-llvm"), FILES))
    return {f: (d / f).read_text().splitlines() for f in FILES}


def test_a_barrier_orders_memory_for_the_compiler(ir):
    """LDS stores before a barrier and loads after it stay where they are only if the barrier is one for the compiler too:
    fences on both sides (__syncthreads) or an asm statement that clobbers memory."""
    seen = 0
    for f, lines in ir.items():
        for i, line in enumerate(lines):
            if re.search(r"call void @llvm\.amdgcn\.s\.barrier", line):
                seen += 1
                assert "fence" in lines[i - 1] and "release" in lines[i - 1], (f, lines[i - 2:i + 2])
                assert "fence" in lines[i + 1] and "acquire" in lines[i + 1], (f, lines[i - 2:i + 2])
            elif "s_barrier" in line:
                seen += 1
                assert "~{memory}" in line, (f, line)
    assert seen > 10


def test_direct_to_lds_loads_declare_m0(ir):
    """The LDS address of such a load is passed in m0, which the compiler may be using for something else."""
    asm = [line for lines in ir.values() for line in lines if "asm sideeffect" in line and " lds" in line]
    assert len(asm) > 50
    assert all("~{m0}" in line for line in asm if "m0" in line.split("~{")[0])
