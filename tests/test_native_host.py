"""The library's host code on the CPU: the launches, copies and waits that the calls enqueue, run by a stand-in
runtime (tests/native/fake_hip.h) in the latest order that the waits allow, with plain loops in place of the kernels."""
import os
import shutil
import subprocess

import pytest

from tests.test_gpu_relay_pieces import RESHARD_PIECES, STAGE_PIECES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_22614_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                                reason="g++ or the HIP headers not available")


def _build(exe, flags):
    sources = [os.path.join(CSRC, f) for f in ("plan.cpp", "capi.cpp", "staging.cpp", "reshard.cpp", "relay.cpp",
                                               "moments.cpp")]
    cmd = ["g++", "-std=c++17", *flags, "-Wall", "-Wno-unused-result", "-D__HIP_PLATFORM_AMD__", "-isystem",
           os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "native", "host_check.cpp"), *sources, "-lpthread", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.fixture(scope="module")
def host_check(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("host") / "host_check"),
                  ["-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"])


@pytest.fixture(scope="module")
def host_check_fast(tmp_path_factory):
    return _build(str(tmp_path_factory.mktemp("host") / "host_check_fast"), ["-O2"])


@pytest.mark.parametrize("mode", ["copies", "sums", "destroy", "order"])
def test_host_code(host_check, mode):
    r = subprocess.run([host_check, mode], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert " 0 errors" in r.stdout


@pytest.mark.parametrize("model,w,to,b,depth,pieces", STAGE_PIECES + [(m, w, -w2, b, 0, n) for m, w, w2, b, n in RESHARD_PIECES])
def test_pieces_of_the_path_through_host_memory(host_check_fast, model, w, to, b, depth, pieces):
    """The layouts that the GPU test runs: they are cut into as many pieces as it claims, and put together again."""
    r = subprocess.run([host_check_fast, "pieces", *map(str, (*model, w, to, b, depth))], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert int(r.stdout.split()[1]) == pieces
