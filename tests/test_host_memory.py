"""The library's device allocations, compiled for the host against a simulated
card (tests/host_memory.cpp); no GPU."""
import os
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2306_08252_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("host_memory") / "host_memory")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", "-I", CSRC,
                        os.path.join(ROOT, "tests", "host_memory.cpp"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.mark.parametrize("check", ["scratch_growth_fails"])
def test_device_memory(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
