"""The row tiles that one LP's own launches take: the tuned shape where its tiles fill the device, a
smaller one where they do not, a larger one where a tile holds few rows; and the same results
whichever it is."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu


def _lp(m, n, row, seed=0):
    """`row` entries in every row, about m * row / n in every column."""
    rng = np.random.default_rng([m, n, row, seed])
    keys = np.unique(np.repeat(np.arange(m, dtype=np.int64) * n, row) + rng.integers(0, n, size=m * row))
    return synth.kkt_constructed(m, n, keys, rng, eq_frac=0.4, name=f"{m}x{n} {row}")


def _run(lp, **opts):
    with lpg.Solver(lp, method=1, eps_rel=0.0, max_iters=70, small_lp_lds=0, **opts) as s:
        sol = s.solve()
        return s.layout(), [sol.x, sol.y, sol.z, *s.iterates(), np.array([sol.info.rel_kkt, sol.info.restarts])]


@pytest.mark.parametrize("precision,tuned", [(0, 1024), (1, 2048)])
def test_short_rows(precision, tuned):
    lp = _lp(120000, 180000, 11)
    lay, got = _run(lp, spmv_layout=1, precision=precision)
    print(lay, flush=True)
    assert lay["tile_nnz"] == tuned
    assert (lay["flat_a"], lay["flat_at"]) == (lay["tiles_a"], lay["tiles_at"])
    _, want = _run(lp, spmv_layout=1, precision=precision, tile_nnz=tuned)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("precision", [0, 1])
def test_few_tiles_and_few_rows_in_a_tile(precision):
    few = _lp(20000, 30000, 11)
    lay, _ = _run(few, spmv_layout=1, precision=precision)
    assert lay["tile_nnz"] > 1024 and lay["flat_a"] > 1.8 * lay["tiles_a"]
    long_rows = _lp(4999, 9998, 205)  # above 7/8 of a 4096-entry tile for each of 256 CUs
    lay, got = _run(long_rows, spmv_layout=1, precision=precision)
    assert lay["tile_nnz"] < 4096 and lay["flat_a"] < 0.6 * lay["tiles_a"]
    _, want = _run(long_rows, spmv_layout=1, precision=precision, tile_nnz=lay["tile_nnz"])
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("row", [400, 1300])
def test_rows_that_a_workgroup_reduces(row, precision):
    """All rows longer than long_row_len, in the panel layout: as in the panels themselves."""
    lp = _lp(900, 6000, row)
    lay, got = _run(lp, precision=precision)
    assert lay["long_rows_a"] == 900 and lay["flat_a"] == 900
    _, want = _run(lp, precision=precision, panel_slice_bytes=8 * 3001)
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a, b)
