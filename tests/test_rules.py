"""CPU check of the rules that choose launches and kernels (no device needed):
compiles tests/rules_harness.cpp against the built library and runs it."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1810_02612_amd")


def test_rules(tmp_path):
    if not os.path.exists(os.path.join(PKG, "liblbl.so")):
        pytest.skip("library not built")
    exe = str(tmp_path / "harness")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                           os.path.join(ROOT, "tests", "rules_harness.cpp"), "-L", PKG, "-llbl",
                           f"-Wl,-rpath,{PKG}", "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    assert "rules OK" in r.stdout
