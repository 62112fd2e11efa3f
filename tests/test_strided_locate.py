"""The compact 32-bit program that the chunk kernels locate with against the general layout program, on the host."""
import os
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2402_12274_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")


def test_compact_program_equals_general_program():
    if not os.path.isdir("/opt/rocm/include"):
        pytest.skip("HIP headers not installed")
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "strided_check")
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I",
                               os.path.join(ROOT, "include"), "-I", CSRC,
                               *[os.path.join(CSRC, s) for s in ("types.cpp", "compile.cpp", "trace.cpp")],
                               os.path.join(NATIVE, "host_stub.cpp"), os.path.join(NATIVE, "strided_check.cpp"), "-o", exe,
                               "-lpthread", "-ldl"])
        r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        assert "bad 0" in r.stdout
