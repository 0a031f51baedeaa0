"""The device memory kept between calls (csrc/ftle_memory.h), on the CPU: its
code is compiled against a pretend device (kept_memory.cpp)."""
import os
import subprocess

import pytest

from paper_2408_02758_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("kept") / "kept_memory")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-function", "-D__HIP_PLATFORM_AMD__",
                    "-I", B.CSRC, "-I", os.path.join(rocm, "include"), os.path.join(HERE, "kept_memory.cpp"),
                    "-o", exe, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("check", ["out_of_memory", "failed_wait", "bound"])
def test_kept_memory(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
