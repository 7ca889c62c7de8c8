"""What the passes write stays inside the buffer that the plan gave it: every pass and operator of a handle is run without a
GPU (tests/emu/scratch_check.cpp), and the slices of every split reduction have to lie inside one buffer of the workspace."""
import os
import shutil
import subprocess

import pytest

import synthetic_inputs as S

HERE = os.path.dirname(os.path.abspath(__file__))
PACKAGE = os.path.join(os.path.dirname(HERE), "paper_1412_2302_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def line(wl, batch, precision, flags=0):
    conv = [v for layer in wl["conv"] for v in layer]
    return " ".join(map(str, [batch, wl["in_c"], wl["crop"], wl["crop"], wl["raw"], wl["raw"], *conv, *wl["fc"],
                              precision, flags]))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_slices_stay_inside_their_buffers(tmp_path):
    from paper_1412_2302_amd import build
    lib = build.LIB if os.path.exists(build.LIB) else build.build(verbose=False)
    exe, cases = str(tmp_path / "scratch_check"), tmp_path / "cases"
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"), "-rdynamic",
                    "-o", exe, os.path.join(HERE, "emu", "scratch_check.cpp"), lib, "-Wl,-rpath," + PACKAGE], check=True,
                   timeout=900)
    # every batch up to 64 and from there on every 13th to 2048: the lines between kernels and slice counts lie anywhere
    batches = [*range(1, 65), *range(65, 2049, 13)]
    cases.write_text("\n".join(line(wl, b, precision, flags) for wl in S.WORKLOADS.values() for b in batches
                               for precision, flags in ((0, 0), (1, 0), (0, 1))) + "\n")
    # dense layers that start between quads behind one another, in vectors whose ends do not
    with cases.open("a") as f:
        for wl, fc in ((wl, fc) for wl in S.WORKLOADS.values() for fc in ((3, 5, 1), (201, 135, 35), (5, 512, 4), (64, 7, 12))):
            for b in (1, 2, 4, 7, 8, 16, 37, 64, 200):
                f.write("\n".join(line(dict(wl, fc=fc), b, precision) for precision in (0, 1)) + "\n")
    r = subprocess.run([exe, str(cases), "7", "6000"], capture_output=True, text=True, timeout=1500)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-2000:]
    assert r.stdout.rstrip().endswith(" 0 outside")
