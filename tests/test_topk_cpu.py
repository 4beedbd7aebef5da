"""The top-k kernels compiled for the CPU (tests/cpu_hip, tests/topk_cpu.cpp):
calls that overlap on one scratch stay inside their buffers."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs clang++")
def test_overlapping_calls_stay_in_bounds(tmp_path):
    exe = str(tmp_path / "topk_cpu")
    r = subprocess.run([CLANG, "-std=c++17", "-O1", "-I", os.path.join(HERE, "cpu_hip"),
                        os.path.join(HERE, "topk_cpu.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout[-500:])
