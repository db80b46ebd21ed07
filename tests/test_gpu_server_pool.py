"""A server's requests set up by several threads in memory that earlier requests gave back:
repeated rounds of requests of very different sizes, under a budget that makes them wait and
one that does not, give the solo results and stay within the budget."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu
OPTS = dict(spmv_layout=1, method=1, precision=1, eps_rel=0.0, max_iters=192)


@pytest.mark.parametrize("tight", [True, False])
def test_rounds_of_requests(tight):
    rng = np.random.default_rng(11)
    lps = [synth.cfg0(0), synth.cfg4_lp(3, m_hi=3000), synth.transportation(300, rng), synth.cfg4_lp(5, m_hi=800),
           synth.cfg1(0, m=6000, n=12000, nnz=70000), synth.cfg0(1)]
    solo = []
    for lp in lps:
        with lpg.Solver(lp, small_lp_lds=0, **OPTS) as s:
            solo.append(s.solve())
    templates = [lpg.Solver(lp, deferred=1, **OPTS) for lp in lps]
    sizes = [t.layout()["device_bytes"] for t in templates]
    budget = int(1.3 * max(sizes)) if tight else 1 << 33
    try:
        with lpg.Server(budget, 4, **OPTS) as srv:
            for r in range(4):
                order = rng.permutation(len(lps))
                print("round", r, order.tolist(), flush=True)
                tickets = [(i, srv.submit(templates[i])) for i in order]
                srv.wait(60.0)
                for i, t in tickets:
                    got = srv.result(t)
                    assert got.info.iterations == 192
                    np.testing.assert_array_equal(got.x, solo[i].x)
                    np.testing.assert_array_equal(got.y, solo[i].y)
            st = srv.stats()
            assert st["peak_bytes"] <= budget and st["bytes_in_use"] == 0 and st["completed"] == 4 * len(lps)
    finally:
        for t in templates:
            t.close()
