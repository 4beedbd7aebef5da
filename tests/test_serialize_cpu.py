"""The serialisation kernel compiled for the CPU (tests/cpu_hip,
tests/serialize_cpu.cpp): every form against a token-by-token reference, inside
its buffers."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs clang++")
def test_every_form_against_a_reference(tmp_path):
    exe = str(tmp_path / "serialize_cpu")
    r = subprocess.run([CLANG, "-std=c++17", "-O1", "-I", os.path.join(HERE, "cpu_hip"),
                        os.path.join(HERE, "serialize_cpu.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", (r.returncode, r.stdout[-500:])
