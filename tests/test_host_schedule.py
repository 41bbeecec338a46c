"""What the host side of the library launches, in which order, and what it
captures, on a machine without a GPU.

Compiles ``csrc/ssfm.cpp`` and links it with ``tests/host/schedule.cpp``, which
stands in for the HIP runtime and the kernels (they compute nothing) and
holds the checks.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_15678_amd", "csrc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    out = tmp_path_factory.mktemp("schedule")
    sources = [os.path.join(CSRC, "ssfm.cpp"), os.path.join(ROOT, "tests", "host", "schedule.cpp")]
    objects = [str(out / (os.path.basename(s) + ".o")) for s in sources]
    exe = str(out / "schedule")
    steps = [[hipcc, "--offload-arch=gfx950", "-O1", "-g", "-std=c++20", "-I",
              os.path.join(ROOT, "include"), "-I", CSRC, "-c", s, "-o", o]
             for s, o in zip(sources, objects)]
    steps.append([hipcc, "--offload-arch=gfx950", *objects, "-o", exe])
    for cmd in steps:
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, " ".join(cmd) + "\n" + r.stdout + r.stderr
    return exe


@pytest.mark.parametrize("check", ["captured", "samples", "graphs", "planes", "entries", "create"])
def test_schedule(program, check):
    r = subprocess.run([program, check], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stdout + r.stderr
