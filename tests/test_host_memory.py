"""What the host runtime does when device memory runs short, on a stub of the HIP API whose
device has bounded memory (tests/host_memory_check.cpp), under AddressSanitizer and
UndefinedBehaviorSanitizer.  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++") or shutil.which("clang++")


@pytest.mark.skipif(CXX is None, reason="no host C++ compiler")
def test_runtime_short_of_memory(tmp_path):
    exe = str(tmp_path / "host_memory_check")
    cmd = [CXX, "-std=c++17", "-O1", "-g", "-Wno-unused-function", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-fno-omit-frame-pointer",
           "-I" + os.path.join(ROOT, "tests", "hoststub_memory"), "-I" + os.path.join(ROOT, "include"),
           "-I" + os.path.join(ROOT, "paper_2305_03945_amd", "csrc"),
           os.path.join(ROOT, "tests", "host_memory_check.cpp"),
           os.path.join(ROOT, "paper_2305_03945_amd", "csrc", "runtime.cpp"), "-o", exe]
    b = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert b.returncode == 0, b.stdout
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300, env=env)
    assert r.returncode == 0 and "host memory checks passed" in r.stdout, r.stdout
