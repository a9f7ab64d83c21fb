"""The library's device-memory bookkeeping on a pretended device (CPU only).

tests/sanitize/memory_driver.cpp runs csrc/buffers.h and csrc/devstore.h
against allocators that can run out, with several threads, under
AddressSanitizer and UndefinedBehaviorSanitizer and under ThreadSanitizer.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
CSRC = os.path.join(ROOT, "paper_1804_02297_amd", "csrc")

pytestmark = pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm clang++ not available")


def _run(tmp_path, name, flags, env):
    exe = str(tmp_path / name)
    r = subprocess.run([CLANG, "-std=c++17", "-O1", "-g", "-pthread", "-Wall", "-I" + CSRC] + flags +
                       [os.path.join(ROOT, "tests", "sanitize", "memory_driver.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, env=dict(os.environ, **env), timeout=120)
    print(r.stdout[-3000:])
    assert r.returncode == 0 and "ALL OK" in r.stdout, r.stderr[-3000:]
    return r


def test_under_address_and_undefined_behaviour_sanitizers(tmp_path):
    r = _run(tmp_path, "memory_asan", ["-fsanitize=address,undefined", "-fno-sanitize-recover=undefined"],
             {"ASAN_OPTIONS": "detect_leaks=1"})
    assert "runtime error" not in r.stderr and "ERROR: AddressSanitizer" not in r.stderr


def test_under_thread_sanitizer(tmp_path):
    r = _run(tmp_path, "memory_tsan", ["-fsanitize=thread"], {})
    assert "ThreadSanitizer" not in r.stderr, r.stderr[-3000:]
