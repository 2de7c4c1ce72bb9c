"""What libmg launches, checked without a GPU: tests/host/launch_sim.cpp is
linked against the built library and stands in for the HIP runtime, recording
each launch (kernel, grid, arguments) instead of enqueueing it."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1602_08477_amd")
LIB = os.path.join(PKG, "libmg.so")
CLANGXX = "/opt/rocm/lib/llvm/bin/clang++"

pytestmark = pytest.mark.skipif(not os.path.exists(CLANGXX) and not shutil.which("g++"),
                                reason="needs a C++ compiler")


def test_host_launches(tmp_path):
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} is missing: build() makes it")
    exe = str(tmp_path / "launch_sim")
    cxx = CLANGXX if os.path.exists(CLANGXX) else "g++"
    r = subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-rdynamic",
                        "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "host", "launch_sim.cpp"), "-o", exe,
                        "-L" + PKG, "-lmg", "-Wl,-rpath," + PKG, "-L/opt/rocm/lib",
                        "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64", "-ldl"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    assert "0 failures" in r.stdout
