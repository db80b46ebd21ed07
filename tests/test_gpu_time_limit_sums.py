"""The statistics that a time-limited lp_solve on one workgroup returns are the ones its stop was
decided on: those of the last trace record, above eps_rel exactly when the status says so, and
the oracle's index-order sums of the returned point, from both one-workgroup kernels."""
import numpy as np
import pytest

import oracle
import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu


def _long_row():
    rng = np.random.default_rng(4)
    keys = np.concatenate([np.arange(129)] + [i * 300 + np.sort(rng.choice(300, 4, replace=False)) for i in range(1, 80)])
    return synth.kkt_constructed(80, 300, keys.astype(np.int64), rng, name="a row of 129 entries")


def _cases():
    return [(synth.cfg0(0), 1), (synth.transportation(150, np.random.default_rng(6)), 1), (_long_row(), 2)]


@pytest.mark.parametrize("eps", [0.0, 1e-9])
@pytest.mark.parametrize("method", [0, 1])
@pytest.mark.parametrize("i", range(3))
def test_returned_statistics_are_the_decided_ones(oracle_lib, i, method, eps):
    lp, solver = _cases()[i]
    for limit in (1e-7, 1e-3, 0.02):
        print(lp.name, method, limit, flush=True)
        with lpg.Solver(lp, spmv_layout=1, method=method, eps_rel=eps, max_iters=10**7, time_limit_s=limit,
                        trace_cap=100000) as s:
            sol = s.solve(with_trace=True)
            assert s.layout()["last_solver"] == solver and sol.info.solve_path == 1
        info, last = sol.info, sol.trace[-1]
        assert sol.status in ("time_limit", "optimal")
        assert (info.rel_kkt <= eps) == (sol.status == "optimal")
        if sol.status == "optimal":
            continue
        assert last[0] == info.iterations
        assert info.rel_kkt == last[5 if info.output_is_avg else 4]
        chk = oracle.kkt(lp, sol.x, sol.y)
        assert (info.primal_obj, info.dual_obj) == (chk["pobj"], chk["dobj"])
