"""The tables of the core kernels (host_cores.cpp) built with g++ under AddressSanitizer and UndefinedBehaviorSanitizer,
without device code, and checked against the operators (tests/native/core_tables.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1801_08432_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_core_tables_under_asan_and_ubsan(tmp_path):
    exe = str(tmp_path / "core_tables")
    srcs = [os.path.join(ROOT, "tests", "native", "core_tables.cpp")] + [
        os.path.join(CSRC, f) for f in ("host_basis.cpp", "host_cores.cpp")]
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=undefined", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe] + srcs
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0:verify_asan_link_order=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "runtime error" not in r.stderr and "AddressSanitizer" not in r.stderr, r.stderr
    assert "0 failed" in r.stdout
