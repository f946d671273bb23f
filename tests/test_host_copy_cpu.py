"""Copies between pageable host arrays and the device, on the CPU.

`tests/sanitizer/copy_driver.hip` defines the HIP runtime calls that `csrc/host_copy.hip` makes (a
copy is a memcpy) and is built with it as the host pass of a HIP compile, under ThreadSanitizer.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "sanitizer")
CSRC = os.path.join(ROOT, "paper_2112_01975_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("copy") / "copy_driver")
    cmd = [HIPCC, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-g", "-I", CSRC, "-Xarch_host", "-fsanitize=thread",
           os.path.join(HERE, "copy_driver.hip"), os.path.join(CSRC, "host_copy.hip"), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True)
    return exe


@pytest.mark.parametrize("check", ["data", "worth_the_threads", "quota", "per_thread_stream", "current_device", "block", "block_to_device", "no_pinned_memory", "capture_mode"])
def test_copies_through_worker_threads(driver, check):
    r = subprocess.run([driver, check], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "copy driver ok" in r.stdout, (r.stdout + r.stderr)[-4000:]
