"""CPU check of the run encoding and its tilings (no device needed): compiles
tests/run_layout_harness.cpp against the built library and runs it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1810_02612_amd")


def test_run_codes_and_tilings(tmp_path):
    if not os.path.exists(os.path.join(PKG, "liblbl.so")):
        pytest.skip("library not built")
    exe = str(tmp_path / "harness")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                           os.path.join(ROOT, "tests", "run_layout_harness.cpp"), "-L", PKG, "-llbl",
                           f"-Wl,-rpath,{PKG}", "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    assert "run layout OK" in r.stdout
