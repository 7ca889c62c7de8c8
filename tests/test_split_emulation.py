"""Builds and runs the CPU emulation of the three-term fp32 products (csrc/gemm_split.h): exactness of the split, and
loaders, LDS layout, fragment maps and epilogues against double-precision loops, under sanitizers.  No GPU involved."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_split_workgroup_program_on_cpu(tmp_path):
    exe = str(tmp_path / "split_emu")
    src = os.path.join(HERE, "emu", "split_emu.cpp")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-o", exe, src], check=True, timeout=900)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=900)
    assert r.returncode == 0, r.stdout[-3000:] + r.stderr[-3000:]
    assert "ALL OK" in r.stdout and "FAIL" not in r.stdout
