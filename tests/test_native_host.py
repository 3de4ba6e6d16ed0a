"""The library's host code on the CPU: the launches, copies and waits that the calls enqueue, run by a stand-in
runtime (tests/native/fake_hip.h) in the latest order that the waits allow, with plain loops in place of the kernels."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_22614_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                                reason="g++ or the HIP headers not available")


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_check")
    sources = [os.path.join(CSRC, f) for f in ("plan.cpp", "capi.cpp", "staging.cpp", "reshard.cpp", "relay.cpp",
                                               "moments.cpp")]
    cmd = ["g++", "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall",
           "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(ROCM, "include"), "-I",
           os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "native", "host_check.cpp"), *sources,
           "-lpthread", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("mode", ["copies", "sums", "destroy", "order"])
def test_host_code(host_check, mode):
    r = subprocess.run([host_check, mode], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert " 0 errors" in r.stdout
