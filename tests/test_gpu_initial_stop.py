"""A solve that stops at its initial point: the iterates are that point, in both precisions and from
every solver. The FP32 form adds its corrections to a master point; both were left as they lay
in memory, which an earlier handle of the same size had used."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu


def _lps(m, n):
    """Two LPs of one size: one to be solved, one whose initial point 0 is optimal (c >= 0, 0 feasible)."""
    rng = np.random.default_rng([m, n])
    keys = np.unique(np.concatenate((rng.integers(0, m * n, size=3 * n), np.arange(m) * np.int64(n))))
    lp = synth.kkt_constructed(m, n, keys.astype(np.int64), rng, eq_frac=0.0)
    done = synth.LP(m, n, lp.row_ptr, lp.col_idx, lp.vals, np.abs(lp.c) + 1.0, np.full(m, -np.inf), np.full(m, 5.0),
                    np.zeros(n), np.full(n, 9.0))
    return lp, done


CALLS = {
    "one workgroup": lambda s, o: s.solve(),
    "kernel loop": lambda s, o: s.solve_until(10**6),
    "batch": lambda s, o: lpg.solve_batch([s], batch_split_nnz=1 << 40, **o)[0],
    "batch, row tiles": lambda s, o: lpg.solve_batch([s], batch_split_nnz=1 << 40, small_lp_lds=0, **o)[0],
    "block diagonal": lambda s, o: lpg.solve_batch([s], batch_split_nnz=0, **o)[0],
}


@pytest.mark.parametrize("method", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("call", list(CALLS))
def test_iterates_are_the_initial_point(call, precision, method):
    for m, n in ((1, 7), (60, 130), (700, 1500)):
        lp, done = _lps(m, n)
        opts = dict(method=method, precision=precision, spmv_layout=1)
        for eps, iters, p in ((0.0, 200, lp), (0.0, 200, done)):
            print(call, m, n, p is done, flush=True)
            with lpg.Solver(p, eps_rel=eps, max_iters=iters, **opts) as s:
                sol = CALLS[call](s, dict(eps_rel=eps, max_iters=iters, method=method))
                its = s.iterates()
        assert sol.status == "optimal" and sol.info.iterations == 0
        for v in (*its, sol.x, sol.y):
            assert not v.any(), (m, n)
