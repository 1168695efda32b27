"""Host check of the byte moduli's FP64 CRT sum (crt_bytes.hpp), on the CPU:
compiled with g++ together with tests/host/crt_check.cpp, which compares
every result it claims with the 128-bit integer rounding."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_09095_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "host", "crt_check.cpp")


def test_crt_sum_never_departs_from_exact(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path / "crt_check")
    cmd = [gxx, "-O2", "-std=c++20", "-ffp-contract=off", "-D__device__=", "-D__forceinline__=inline",
           "-D__mul24(a,b)=((a)*(b))", f"-I{CSRC}", "-o", exe, SRC]
    build = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout + run.stderr
    assert "mismatches 0" in run.stdout
