"""Host check of the server's memory pool (lp_server_pool.h): `server_pool_check.cpp` runs it over a
memory that records every allocation, release and wait."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_23951_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_server_pool(tmp_path):
    exe = str(tmp_path / "server_pool_check")
    cxx = os.environ.get("HOST_CXX", "g++").split()
    r = subprocess.run([*cxx, "-O1", "-g", "-std=c++17", "-Wall", "-pthread", "-I", CSRC, "-o", exe,
                        os.path.join(HERE, "server_pool_check.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
