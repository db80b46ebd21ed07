"""Row tiles of matrices on both sides of the bound on plain loads (370 MB an iteration in a
solve of its own, 430 MB over all FP64 LPs of block-diagonal launches): the loads differ, the
results do not. A solve of its own is compared with a tile shape that was asked for and with its
block-diagonal solve; block-diagonal solves alone (plain loads) and together (non-temporal)."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu


def _lp(m, n, row, seed):
    rng = np.random.default_rng([m, n, seed])
    keys = np.unique(np.repeat(np.arange(m, dtype=np.int64) * n, row) + rng.integers(0, n, size=m * row))
    return synth.kkt_constructed(m, n, keys, rng, free_frac=0.2, eq_frac=0.35, two_sided_frac=0.3, name=f"{m}x{n}")


def _bytes(lp, value):
    """What an iteration streams: entries of both matrices, vectors twice."""
    return 2 * lp.nnz * (value + 4) + 2 * value * (9 * lp.n + 8 * lp.m)


def _own(lp, **opts):
    with lpg.Solver(lp, spmv_layout=1, eps_rel=0.0, max_iters=40, **opts) as s:
        sol = s.solve()
        assert s.layout()["last_solver"] == 0
        return [sol.x, sol.y, sol.z, *s.iterates(), np.array([sol.info.rel_kkt, sol.info.restarts])]


def _together(lps, **opts):
    solvers = [lpg.Solver(lp, spmv_layout=1, **opts) for lp in lps]
    try:
        sols = lpg.solve_batch(solvers, eps_rel=0.0, max_iters=40, batch_split_nnz=0,
                               **{k: v for k, v in opts.items() if k == "method"})
        return [[s.x, s.y, s.z, *h.iterates(), np.array([s.info.rel_kkt, s.info.restarts])] for s, h in zip(sols, solvers)]
    finally:
        for s in solvers:
            s.close()


def _equal(a, b):
    for u, v in zip(a, b):
        np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("method", [0, 1])
@pytest.mark.parametrize("row", [11, 13])
def test_own_launches(row, method):
    lp = _lp(600000, 1000003, row, 1)
    assert (_bytes(lp, 8) > 370 << 20) == (row == 13)
    got = _own(lp, method=method)
    print(lp.nnz, method, flush=True)
    _equal(got, _own(lp, method=method, tile_nnz=1024))
    _equal(got, _together([lp], method=method)[0])


@pytest.mark.parametrize("precision", [0, 1])  # (FP32: plain loads on both sides)
def test_block_diagonal_launches(precision):
    lps = [_lp(150000 + 501 * i, 250003, 12 + i, i) for i in range(6)]
    total = sum(_bytes(lp, (8, 4)[precision]) for lp in lps) * (1, 2)[precision]
    assert total > 430 << 20 > max(_bytes(lp, 8) for lp in lps)
    alone = [_together([lp], method=1, precision=precision)[0] for lp in lps]
    print(precision, total >> 20, flush=True)
    for i, got in enumerate(_together(lps * (1, 2)[precision], method=1, precision=precision)):
        _equal(got, alone[i % len(lps)])
