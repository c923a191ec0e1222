"""The library's host code over a HIP runtime of the test's own (tests/fake_runtime.cpp, no GPU):
what it does when device memory runs out, what it keeps, and what a call does after another.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = ["tests/fake_runtime.cpp"] + [f"paper_1008_2410_amd/csrc/{f}.cpp"
                                        for f in ("api", "adaptive", "device_cache", "tables", "host_tree")]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("fake_runtime")
    objects = [str(d / (os.path.basename(s) + ".o")) for s in SOURCES]
    jobs = [subprocess.Popen([hipcc, "-w", "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-c", s, "-o", o],
                             cwd=ROOT) for s, o in zip(SOURCES, objects)]
    assert all(j.wait() == 0 for j in jobs)
    exe = str(d / "fake_runtime")  # linked without the HIP runtime
    subprocess.run(["g++", *objects, "-o", exe, "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("check", ["call_memory", "warm_calls", "held_memory", "idle_released",
                                   "host_memory", "work_order", "shared_workspace"])
def test_host_runtime(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and f"{check} passed" in r.stdout, r.stdout[-3000:] + r.stderr[-1000:]
