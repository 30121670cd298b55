"""A reverse pass that memory allows in its one-launch form is not refused
because the form whose recomputes share launches was tried first: the C ABI's
host code runs against a stand-in HIP runtime with a byte budget
(tests/host/memory_driver.cpp), on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_reverse_pass_with_little_memory(tmp_path):
    csrc = os.path.join(ROOT, "paper_1101_0086_amd", "csrc")
    exe = str(tmp_path / "memory_driver")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
                    os.path.join(csrc, "mpa_api.cpp"), os.path.join(ROOT, "tests", "host", "memory_driver.cpp"),
                    "-o", exe], check=True, capture_output=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0 and "OK (0 failures)" in r.stdout, (r.stdout + r.stderr)[-3000:]
