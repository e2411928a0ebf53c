"""The scatter pass turns each group's sum into a 64-bit integer: exactly, whatever its
sign or size, and 0 where it is not a number or infinite."""
import os
import subprocess

import pytest

from tests.test_host_emulation import CLANG, CSRC, EMU, ROOT


def run_program(tmp_path, source, *more):
    """Compile one host program of tests/hostemu (and more sources beside it) with the kernels' headers and run it."""
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ is not installed")
    exe = str(tmp_path / "program")
    # the kernels' helpers that the program does not call stay undefined
    cmd = [CLANG, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-DVCT_HOST_EMULATION", "-I/opt/rocm/include",
           f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", f"-I{EMU}", "-include", "emu.h", "-include", "cfloat",
           "-fsanitize=undefined,float-cast-overflow", "-fno-sanitize-recover=all", "-Wno-unused-value",
           "-Wno-unused-function", *(os.path.join(EMU, f) for f in (source, *more)), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


def test_fixed_point_is_the_rounded_product(tmp_path):
    run_program(tmp_path, "fixed_point_case.cpp")
