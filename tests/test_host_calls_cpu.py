"""What the library's host code enqueues and how long the host memory behind it lives (no GPU):
tests/sanitize/host_calls.cpp compiles tc_host.cpp against the runtime of tests/sanitize/fake_hip.h,
with AddressSanitizer and UndefinedBehaviorSanitizer, and runs one check per test."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
SAN = ["-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]
ENV = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:halt_on_error=1",
           UBSAN_OPTIONS="print_stacktrace=1:halt_on_error=1")
CHECKS = ["gradient_order", "image_streams", "image_capture", "pageable_capture", "launch_limits", "adjoint_tile"]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip")),
                                reason="no g++ or HIP headers")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host_calls") / "host_calls")
    r = subprocess.run(["g++", *SAN, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1002_1050_amd", "csrc"),
                        "-o", exe, os.path.join(ROOT, "tests", "sanitize", "host_calls.cpp"), "-lpthread"],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.mark.parametrize("check", CHECKS)
def test_host_calls(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=300, env=ENV)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-4000:] + r.stderr[-4000:]
