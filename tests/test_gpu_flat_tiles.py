"""Row tiles of one LP's own launches, in place of the panel units where the gathered vector is
short and in place of the tuned shape in the row-tile layout: the same iterates, bit for bit,
as the panels (a panel width that was asked for is kept) and as a tile shape that was asked
for, with rows that a workgroup reduces (over long_row_len, or over a tile) among them."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu


def _lp(m, n, lengths, seed):
    rng = np.random.default_rng([m, n, seed])
    k = rng.integers(1, 6, size=m)
    for row, length in lengths:
        k[row] = length
    keys = np.concatenate([i * n + np.sort(rng.choice(n, size=min(int(q), n), replace=False)) for i, q in enumerate(k)])
    return synth.kkt_constructed(m, n, keys.astype(np.int64), rng, eq_frac=0.5, name=f"{m}x{n}")


CASES = {
    "short rows": (700, 1400, [], {}),
    "one row, one tile": (1, 7, [], {}),
    "rows at the long-row length": (600, 3000, [(0, 256), (3, 257), (599, 300)], {}),
    "rows beyond every tile": (500, 9000, [(7, 5000), (8, 4096), (9, 4097), (490, 1025)], {}),
    "a long-row length above the tiles": (500, 9000, [(7, 5000), (8, 4400)], dict(long_row_len=4500)),
    "a long-row length between two tiles": (500, 9000, [(7, 1500), (8, 1999), (9, 2001)], dict(long_row_len=2000)),
    "many tiles": (90000, 60000, [(5, 900), (80000, 256)], {}),
}


def _iterates(lp, **opts):
    with lpg.Solver(lp, eps_rel=0.0, max_iters=130, small_lp_lds=0, **opts) as s:
        sol = s.solve()
        assert sol.info.solve_path == 0
        return [*s.iterates(), sol.x, sol.y, sol.z, np.array([sol.info.restarts, sol.info.rel_kkt])]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("method", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_tiles_equal_panels(name, method, precision):
    m, n, lengths, opts = CASES[name]
    lp = _lp(m, n, lengths, 3)
    print(name, method, precision, flush=True)
    want = _iterates(lp, method=method, precision=precision, panel_slice_bytes=8 * (max(m, n) // 2 + 1), **opts)
    got = _iterates(lp, method=method, precision=precision, **opts)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["short rows", "one row, one tile", "rows at the long-row length", "many tiles"])
def test_tiles_equal_the_tuned_shape(name, precision):
    m, n, lengths, _ = CASES[name]
    lp = _lp(m, n, lengths, 4)
    opts = dict(method=1, precision=precision, spmv_layout=lpg.LP_LAYOUT_TILES)
    with lpg.Solver(lp, max_iters=0, **opts) as s:
        shape = s.layout()["tile_nnz"]
    for a, b in zip(_iterates(lp, **opts), _iterates(lp, tile_nnz=shape, **opts)):
        np.testing.assert_array_equal(a, b)
