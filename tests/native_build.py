"""Builds the native CPU checks under tests/native with g++ and the HIP headers (no HIP runtime, no GPU)."""
import os
import shutil
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_22614_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
MISSING = shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip"))
SANITIZE = ("-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all")


def native(exe, check, sources=(), flags=SANITIZE):
    """Compiles tests/native/<check> with csrc/<sources> to the program exe."""
    cmd = ["g++", "-std=c++17", *flags, "-Wall", "-Wno-unused-result", "-Wno-attributes", "-D__HIP_PLATFORM_AMD__", "-isystem",
           os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           os.path.join(ROOT, "tests", "native", check), *[os.path.join(CSRC, f) for f in sources], "-lpthread", "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def run(exe, *args):
    """Runs a check; returns what it printed."""
    r = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert " 0 errors" in r.stdout
    return r.stdout
