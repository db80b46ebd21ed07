"""Device memory of a server without requests: what its pool may keep (an eighth of the budget and
256 MB at most), not the footprints of the requests it has completed."""
import time

import numpy as np
import pytest
import torch

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu


def test_an_idle_server_gives_its_memory_back():
    opts = dict(spmv_layout=1, method=1, precision=1, eps_rel=0.0, max_iters=64)
    lp = synth.cfg1(0, m=60000, n=120000, nnz=1400000)
    with lpg.Solver(lp, deferred=1, **opts) as t:
        size = t.layout()["device_bytes"]
        budget = 6 * size
        kept = min(budget // 8, 256 << 20)
        with lpg.Server(budget, 8, **opts) as srv:
            for r in range(2):
                before = torch.cuda.mem_get_info(0)[0]
                tickets = [srv.submit(t) for _ in range(5)]
                srv.wait(60.0)
                points = [srv.result(k).x for k in tickets]
                for x in points[1:]:
                    np.testing.assert_array_equal(x, points[0])
                deadline = time.time() + 10
                while before - torch.cuda.mem_get_info(0)[0] > kept + (64 << 20) and time.time() < deadline:
                    time.sleep(0.02)
                held = before - torch.cuda.mem_get_info(0)[0]
                print(r, size, budget, held, flush=True)
                assert held <= kept + (64 << 20) < 5 * size  # (launch maps and the runtime's own)
