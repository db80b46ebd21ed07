"""Two-phase products (large panel-layout matrices) against the panels, which an explicit panel
width keeps: the same iterates, points and statistics bit for bit, in both forms and precisions,
with long rows (several to a tile), a row longer than a tile, empty rows and columns, and a
last column block and tile that are nearly empty."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu


def _lp(m, n, nnz, long_rows, long_cols, seed):
    rng = np.random.default_rng([m, n, seed])
    keys = [rng.integers(0, m, size=nnz) * n + rng.integers(0, n, size=nnz)]
    for i, k in enumerate(long_rows):
        keys.append((i * 37 % m) * np.int64(n) + rng.integers(0, n, size=k))
    for j, k in enumerate(long_cols):
        keys.append(rng.integers(0, m, size=k) * np.int64(n) + (j * 91 % n))
    keys = np.unique(np.concatenate(keys))
    rows = keys // n
    keys = keys[(rows % 1000 != 999)]  # empty rows
    return synth.kkt_constructed(m, n, keys, rng, free_frac=0.2, eq_frac=0.35, two_sided_frac=0.3, name=f"{m}x{n}")


CASES = {
    # x beyond 4 MB in both precisions, y beyond it in neither; few entries per column block
    "wide": (3000, 1100003, 300000, [300, 257, 9000, 20000], []),
    # both vectors beyond 1.5 MB with 3M entries: both matrices in two phases
    "large": (400001, 800009, 3200000, [256, 257, 5000], [300, 2000, 4999, 8000, 16000]),
    # x just beyond 4 MB in FP64: a last block of one column
    "edge": (70000, 524289, 200000, [], [400]),
}


def _run(lp, **opts):
    with lpg.Solver(lp, eps_rel=0.0, max_iters=70, **opts) as s:
        sol = s.solve()
        return [*s.iterates(), sol.x, sol.y, sol.z, np.array([sol.info.rel_kkt, sol.info.sigma_max, sol.info.restarts])]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_two_phase_equals_panels(name, precision):
    lp = _lp(*CASES[name], 5)
    for method in (0, 1):
        print(name, precision, method, flush=True)
        got = _run(lp, method=method, precision=precision)
        want = _run(lp, method=method, precision=precision, panel_slice_bytes=(1 << 19) - 8)
        for a, b in zip(got, want):
            np.testing.assert_array_equal(a, b)
