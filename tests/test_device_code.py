"""What the compiler makes of the device code (CPU only: every kernel file is compiled for gfx950, nothing is run), and what its
constants are good for."""
import concurrent.futures
import os
import re
import subprocess

import numpy as np
import pytest
from scipy.special import erfc

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
def assembly(tmp_path_factory):
    """Kernels of all files: name -> instructions [(opcode, operands, text)], label -> index; "remarks": what they use."""
    d = tmp_path_factory.mktemp("asm")
    with concurrent.futures.ThreadPoolExecutor(4) as pool:
        remarks = list(pool.map(lambda f: compile_device(f, d / f, "-Rpass-analysis=kernel-resource-usage"), FILES))
    kernels = {"remarks": "".join(remarks)}
    for f in FILES:
        code, labels = None, None
        for line in (d / f).read_text().splitlines():
            line = line.split(";")[0].strip()
            if m := re.match(r"(_Z\w+):$", line):
                kernels[m.group(1)] = code, labels = [], {}
            elif m := re.match(r"([.\w]+):$", line):
                if labels is not None:
                    labels[m.group(1)] = len(code)
            elif line and code is not None and not line.startswith("."):
                op, *rest = line.split(None, 1)
                code.append((op, [a.split()[0] for a in rest[0].split(",")] if rest else [], line))
    return kernels


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


def scalar_registers(operand):
    if m := re.fullmatch(r"s\[(\d+):(\d+)\]", operand):
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.fullmatch(r"s(\d+)", operand)
    return {int(m.group(1))} if m else set()


def test_direct_to_lds_loads_keep_their_distance(assembly):
    """A vector memory instruction may read a scalar register at the earliest five wait states after a vector instruction
    (a lane read of an address or of a spilled register) wrote it.  The compiler inserts waits in its own code, but
    not in front of an asm statement: every path into one is looked at here (s_nop n is n + 1 wait states)."""
    loads = 0
    for name, (code, labels) in ((n, k) for n, k in assembly.items() if n != "remarks"):
        before = [[] for _ in code]
        for i, (op, args, _) in enumerate(code):
            if op.startswith(("s_branch", "s_cbranch")) and labels.get(args[0], len(code)) < len(code):
                before[labels[args[0]]].append(i)
            if op not in ("s_branch", "s_endpgm") and i + 1 < len(code):
                before[i + 1].append(i)
        for i, (op, args, text) in enumerate(code):
            if not (op.startswith("buffer_load") and text.endswith("lds")):
                continue
            loads += 1
            reads = scalar_registers(args[1])
            assert len(reads) == 4, text
            walk, nearest = [(j, 0) for j in before[i]], {}
            while walk:
                j, waits = walk.pop()
                if waits >= 5 or nearest.get(j, 5) <= waits:
                    continue
                nearest[j] = waits
                op_j, args_j, text_j = code[j]
                assert not (op_j.startswith("v_") and args_j and scalar_registers(args_j[0]) & reads), (name, text_j, text, waits)
                walk += [(k, waits + (int(args_j[0], 0) + 1 if op_j == "s_nop" else 1)) for k in before[j]]
    assert loads > 50


def test_no_kernel_spills_vector_registers(assembly):
    """A reload from scratch memory waits for every load in flight: in a loop that streams weights it empties the pipe."""
    names = re.findall(r"Function Name: (\S+)", assembly["remarks"])
    scratch = re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", assembly["remarks"])
    spills = re.findall(r"VGPRs Spill: (\d+)", assembly["remarks"])
    assert len(names) == len(scratch) == len(spills) > 30
    assert not [t for t in zip(names, scratch, spills) if t[1:] != ("0", "0")]


def test_gelu_polynomial_keeps_its_bounds():
    """The exponent polynomial of the bf16 kernels' GELU, with the coefficients as they stand in the source: its largest
    |x (2^p - Q)| where it is fitted, and the largest error of the result in float arithmetic (exponential correctly rounded)."""
    with open(os.path.join(build.CSRC, "group.hpp")) as f:
        body = re.search(r"float gelu_fast\(float z\)\n\{(.*?)\n\}", f.read(), re.S).group(1)
    coef = [np.float32(v) for v in re.findall(r"(-?\d+\.\d+(?:e-\d+)?)f", body.split("float p =")[1].split("const float q")[0])]
    assert len(coef) == 7
    x = np.linspace(0, 5.5, 1 << 20)
    exact = 0.5 * erfc(x / np.sqrt(2))
    assert np.abs(x * (2.0 ** np.polyval(np.float64(coef), x) - exact)).max() < 1.0e-7
    z = np.concatenate([np.linspace(-40, 40, 1 << 21), np.linspace(-9.5, 9.5, 1 << 21), [4.0205336]]).astype(np.float32)
    x = np.abs(z).astype(np.float64)
    c, p = np.clip(x, 0, 9), np.float64(coef[0])
    for k in coef[1:]:
        p = np.float64(np.float32(p * c + np.float64(k)))           # one rounding: the product of two floats is exact
    q = np.exp2(p).astype(np.float32)
    got = np.float32(x * np.float64(np.float32(0.5) - q) + np.float64(np.float32(0.5) * z))
    assert np.abs(got - 0.5 * np.float64(z) * erfc(-np.float64(z) / np.sqrt(2))).max() < 4.0e-7
