"""The layout tuner's shared result: `layout_trial_check.cpp` sets it up from several threads at
once on the host; on the GPU a server does."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2604_23951_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_one_trial_for_concurrent_set_ups(tmp_path):
    exe = str(tmp_path / "layout_trial_check")
    cxx = os.environ.get("HOST_CXX", "g++").split()
    r = subprocess.run([*cxx, "-O1", "-g", "-std=c++17", "-Wall", "-pthread", "-I", CSRC, "-o", exe,
                        os.path.join(HERE, "layout_trial_check.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr


@pytest.mark.gpu
def test_server_sets_up_one_tuned_template_several_times_at_once():
    """Requests of one spmv_layout = 2 template, submitted together and set up on several threads:
    one result for all of them, also for those of a second round."""
    import paper_2604_23951_amd as lpg
    import synth

    lp = synth.cfg4_lp(3, m_hi=3000)
    opts = dict(spmv_layout=2, method=1, eps_rel=0.0, max_iters=128)
    with lpg.Solver(lp, deferred=1, **opts) as t, lpg.Server(1 << 33, 8, **opts) as srv:
        first = None
        for _ in range(2):
            tickets = [srv.submit(t) for _ in range(6)]
            print(tickets, flush=True)
            srv.wait(60.0)
            sols = [srv.result(k) for k in tickets]
            first = first or sols[0]
            for s in sols:
                assert s.info.iterations == 128
                np.testing.assert_array_equal(s.x, first.x)
                np.testing.assert_array_equal(s.y, first.y)
