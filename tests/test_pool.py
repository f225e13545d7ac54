"""The memory kept from closed tables (mlkv_pool.h), checked on the CPU against
a device of the check's own: reuse, the bound on what is kept, that it goes
before an allocation fails, device resets, threads."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2504_01506_amd", "csrc")


def test_kept_memory(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "pool_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wno-deprecated-declarations", "-pthread",
                    "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                    os.path.join(HERE, "pool_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
