"""The serving scheduler's collect threads (csrc/sl_sched.h) against a mock
executor on the CPU: results that take long to fetch hold up no step.  Built
with AddressSanitizer + UBSan and with ThreadSanitizer, host code only."""
import os
import subprocess

import pytest

SRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "sched", "collect_sched.cpp")
CLANG = "/opt/rocm/llvm/bin/clang++"   # (the ThreadSanitizer of g++ 11 reports impossible lock states here)


@pytest.mark.parametrize("compiler,sanitize", [("g++", "address,undefined"), (CLANG, "thread")])
def test_collect_threads(tmp_path, compiler, sanitize):
    if not os.path.exists(compiler) and os.sep in compiler:
        pytest.skip(compiler + " not present")
    exe = str(tmp_path / "collect_sched")
    b = subprocess.run([compiler, "-std=c++17", "-O1", "-g", "-pthread", "-fno-omit-frame-pointer",
                        "-fsanitize=" + sanitize, "-o", exe, SRC], stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True)
    assert b.returncode == 0, b.stdout
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=1", TSAN_OPTIONS="halt_on_error=1"))
    print(r.stdout)
    assert r.returncode == 0 and "0 failure(s)" in r.stdout, r.stdout
