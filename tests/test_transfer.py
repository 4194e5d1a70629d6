"""Read-back of device ranges into the caller's arrays (no GPU: the HIP calls
are stood in for): every chunk arrives, also where allocations fail, a copy
fails, a destination is pinned or the caller's current device is another."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1208_1157_amd", "csrc")
HIP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")


def test_read_back_on_the_cpu(tmp_path):
    if shutil.which("g++") is None or not os.path.isdir(HIP):
        pytest.skip("g++ or the HIP headers are not there")
    exe = str(tmp_path / "transfer_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-I", HIP, "-I",
                    os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "c", "transfer_check.cpp"),
                    os.path.join(CSRC, "fb_transfer.cpp"), "-pthread", "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    got = dict(line.split() for line in out.splitlines())
    assert got == {k: "1" for k in ("plain", "pinned", "device", "errors", "no_memory")}
