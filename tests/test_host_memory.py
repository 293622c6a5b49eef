"""The library's device allocations, compiled for the host against a simulated
card (tests/host_memory.cpp); no GPU."""
import glob
import os
import re
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


@pytest.mark.parametrize("check", ["scratch_growth_fails", "requests_empty_the_cache",
                                   "bounded_and_given_back", "growing_scratch_is_kept",
                                   "error_stays_with_its_call"])
def test_device_memory(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_one_place_allocates():
    """Every device allocation goes through the function that empties the
    cache before it fails."""
    calls = [(os.path.basename(f), line.strip()) for f in sorted(glob.glob(CSRC + "/*"))
             for line in open(f) if re.search(r"\bhipMalloc\(", line)]
    assert calls and {f for f, _ in calls} == {"gv_host.h"}, calls
    assert len(calls) == 2, calls  # the request, and again once the cache is empty


def test_release_without_graphs():
    from paper_2306_08252_amd import graphvine as gv
    if not os.path.exists(gv.LIB_PATH):
        pytest.fail("libgraphvine.so is not built (run __graft_entry__.build())")
    assert gv.gv_release_cached() == 0
