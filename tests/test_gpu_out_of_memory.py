"""Memory that a faster path takes and a solve can do without: an LP that fits the device without the
two-phase layout, or the host without pinned memory for its point, is solved without it. The
allocations are refused in a process of its own, by a host library in front of the runtime's."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.parametrize("child", ["malloc_limit_child.py", "pinned_limit_child.py"])
def test_solved_without_it(child, tmp_path):
    shim = str(tmp_path / "malloc_limit_shim.so")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", shim,
                        os.path.join(HERE, "malloc_limit_shim.cpp"), "-ldl"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([ROOT, HERE]))
    print("child process", child, flush=True)
    r = subprocess.run([sys.executable, os.path.join(HERE, child), shim], env=env, capture_output=True,
                       text=True, timeout=100)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok")
