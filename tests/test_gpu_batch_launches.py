"""Batches whose LPs take several launches (the one-workgroup solver's three sizes, row tiles in LDS
and in global memory): the launches run beside one another, so that with a time limit every LP
gets its time, and every LP's result is its own, whatever launches it meets."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu
SOLO, TILES_LDS, TILES, BLOCK = 1, 2, 3, 4  # lp_get_layout's last_solver


def _random(m, n, nnz, first_row, seed):
    rng = np.random.default_rng([m, n, seed])
    keys = np.concatenate((rng.integers(0, m, size=nnz) * n + rng.integers(0, n, size=nnz), np.arange(first_row),
                           np.arange(m) * n + rng.integers(0, n, size=m)))
    return synth.kkt_constructed(m, n, np.unique(keys).astype(np.int64), rng, name=f"{m}x{n} row {first_row}")


def _lps():
    return [synth.cfg0(0), _random(300, 480, 2000, 0, 1), _random(700, 1400, 5000, 0, 2), _random(80, 300, 300, 129, 3),
            _random(2000, 4000, 80000, 0, 4), _random(60, 200, 200, 0, 5)]


PERSISTENT = [SOLO, SOLO, SOLO, TILES_LDS, TILES, SOLO]


def _solve(lps, call, **opts):
    solvers = [lpg.Solver(lp, spmv_layout=1, method=1) for lp in lps]
    try:
        if call == "static":
            lpg.lp_solve_batch_static([s.h for s in solvers], lpg.make_options(method=1, **opts))
        else:
            lpg.solve_batch(solvers, method=1, batch_split_nnz=1 << 40 if call == "persistent" else 20000, **opts)
        out = []
        for s in solvers:
            x, y, z = np.empty(s.n), np.empty(s.m), np.empty(s.n)
            out.append((lpg.lp_get_solution(s.h, x, y, z), x, y, z, s.layout()["last_solver"]))
        return out
    finally:
        for s in solvers:
            s.close()


@pytest.mark.parametrize("call", ["static", "persistent", "split"])
def test_every_lp_gets_its_time(call):
    lps = _lps()
    print(call, flush=True)
    got = _solve(lps, call, eps_rel=0.0, max_iters=10**7, time_limit_s=0.15)
    assert [g[4] for g in got] == (PERSISTENT if call != "split" else [BLOCK if r == TILES else r for r in PERSISTENT])
    for lp, g in zip(lps, got):
        assert g[0].status == 2 and g[0].iterations >= 256, (lp.name, g[0].iterations)


@pytest.mark.parametrize("count", [6, 300])
@pytest.mark.parametrize("call", ["static", "persistent"])
def test_results_do_not_depend_on_the_launches(call, count):
    """300 LPs (more than the CUs): as many launches as streams, the smaller sizes in wider ones."""
    base = _lps()
    lps = [base[i % len(base)] if i < 12 else base[(0, 5, 1)[i % 3]] for i in range(count)]
    opts = dict(eps_rel=0.0, max_iters=192)
    print(call, count, flush=True)
    alone = [_solve([lp], call, **opts)[0] for lp in base]
    for lp, g in zip(lps, _solve(lps, call, **opts)):
        a = alone[base.index(lp)]
        assert g[4] == a[4] and g[0].rel_kkt == a[0].rel_kkt
        for u, v in zip(g[1:4], a[1:4]):
            np.testing.assert_array_equal(u, v, err_msg=lp.name)
