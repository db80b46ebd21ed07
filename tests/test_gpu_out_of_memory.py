"""An LP that fits the device without the two-phase layout is solved without it: hipMalloc refuses
the larger allocation in a process of its own (a host library in front of the runtime's)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_no_room_for_the_two_phase_layout(tmp_path):
    shim = str(tmp_path / "malloc_limit_shim.so")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", shim,
                        os.path.join(HERE, "malloc_limit_shim.cpp"), "-ldl"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([ROOT, HERE]))
    print("child process", flush=True)
    r = subprocess.run([sys.executable, os.path.join(HERE, "malloc_limit_child.py"), shim], env=env, capture_output=True,
                       text=True, timeout=100)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok")
