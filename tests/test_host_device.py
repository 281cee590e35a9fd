"""CPU checks of the library's host code over memory that stands for a device (host_device.cpp): the
tables that launches are given, and what the handle does where HIP calls fail."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_21794_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("no HIP headers")
    out = str(tmp_path_factory.mktemp("host") / "host_device")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-w", "-D__HIP_PLATFORM_AMD__",
           "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           f"-I{ROCM}/include", f"-I{ROOT}/include", f"-I{CSRC}", "-x", "c++",
           os.path.join(CSRC, "vp_api.cpp"), os.path.join(ROOT, "tests", "host_device.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


CHECKS = ["no_pinned_memory", "large_tables", "failed_upload", "failed_admission"]


@pytest.mark.parametrize("check", CHECKS)
def test_host_code(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]


def test_every_check_is_run(program):
    r = subprocess.run([program], capture_output=True, text=True)
    assert sorted(r.stdout.split()) == sorted(CHECKS)
