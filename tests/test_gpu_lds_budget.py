"""small_lp_lds bounds what the batched solves hold on chip: the solver that runs an LP at every
budget, with the same points. At 0 that is the row tiles in global memory, the reference of the
comparisons with the on-chip solvers."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu
SOLO, TILES_LDS, TILES = 1, 2, 3  # lp_get_layout's last_solver
MAX = 112 * 1024


def _lps():
    rng = np.random.default_rng(9)
    out = [synth.cfg0(0), synth.transportation(400, rng)]
    keys = [np.sort(rng.choice(10000, size=k, replace=False)) + i * 10000 for i, k in enumerate(rng.integers(1, 5, size=5000))]
    out.append(synth.kkt_constructed(5000, 10000, np.concatenate(keys).astype(np.int64), rng, name="5000x10000"))
    return out


def _vectors(lp, precision):
    """Bytes of the vectors that an LP gathers from (each with a zero slot, in whole 16 bytes)."""
    b = 4 if precision else 8
    up = lambda v: (v + 15) // 16 * 16  # noqa: E731
    return max(up(b * (lp.m + 1)) + up(b * (lp.n + 1)), up(8 * (max(lp.m, lp.n) + 1)))


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
def test_solver_at_every_budget(precision, static):
    lps = _lps()
    ref = None
    for budget in (0, 1, 8 * 1024, 40 * 1024, 100 * 1024, MAX - 1, MAX):
        solvers = [lpg.Solver(lp, spmv_layout=1, precision=precision, method=1) for lp in lps]
        opts = dict(eps_rel=0.0, max_iters=64, method=1, small_lp_lds=budget, batch_split_nnz=1 << 40)
        print(precision, static, budget, flush=True)
        try:
            if static:
                lpg.lp_solve_batch_static([s.h for s in solvers], lpg.make_options(**opts))
            else:
                lpg.solve_batch(solvers, **opts)
            ran = [s.layout()["last_solver"] for s in solvers]
            its = [v for s in solvers for v in s.iterates()]
        finally:
            for s in solvers:
                s.close()
        for lp, r in zip(lps, ran):
            if budget == 0:
                assert r == TILES
            elif _vectors(lp, precision) <= budget or budget == MAX:
                assert r == SOLO, (lp.name, budget)
            else:
                assert r in (TILES_LDS, TILES), (lp.name, budget)
        ref = ref or its
        for a, b in zip(its, ref):
            np.testing.assert_array_equal(a, b)
