"""The library's host code on a stand-in HIP runtime (host_calls.hip), without a
GPU: what its calls allocate, wait for, launch and capture."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2603_12016_amd")


@pytest.fixture(scope="module")
def host_calls():
    if not os.path.exists(os.path.join(PKG, "libnyx.so")):
        from paper_2603_12016_amd import build
        build.build()
    exe = os.path.join(ROOT, "tests", "_build", "host_calls")
    os.makedirs(os.path.dirname(exe), exist_ok=True)
    hipcc = "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc"
    tmp = exe + ".tmp%d" % os.getpid()
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-rdynamic",
                           "-I" + os.path.join(PKG, "csrc"), "-I" + os.path.join(ROOT, "include"), "-o", tmp,
                           os.path.join(ROOT, "tests", "host_calls.hip"), "-L" + PKG, "-l:libnyx.so", "-Wl,-rpath," + PKG])
    os.replace(tmp, exe)
    return exe


@pytest.mark.parametrize("check", ["extract_device", "noalloc_wait", "accumulate_wait", "packed_memory",
                                   "band_blocks_of_many", "forks_when_repeated", "plan_counts",
                                   "label_maximum_of_mixed_sizes", "occupancy_of_the_kernel_launched",
                                   "tiles_of_a_box", "tuning_under_a_cap",
                                   "out_of_memory_is_over"])
def test_host_calls(host_calls, check):
    r = subprocess.run([host_calls, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
