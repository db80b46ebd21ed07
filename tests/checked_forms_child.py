"""Solves run by tests/test_gpu_checked_forms.py, in that process with the plain build and in one of
its own with the bounds-checked build (LPGPU_CHECKED=1); there it writes the returned points and the
check word to the .npz file named on the command line."""
import sys

import numpy as np

import paper_2604_23951_amd as lpg
import synth
import test_gpu_two_phase as two_phase


def _empty_slices(m, n, used_rows, used_cols, seed):
    """Entries in the first rows and columns only: the last slices of 64 rows (columns) hold none."""
    rng = np.random.default_rng([m, n, seed])
    cols = [np.sort(rng.choice(used_cols, size=int(k), replace=False)) for k in rng.integers(1, 9, size=used_rows)]
    keys = np.concatenate([i * n + c for i, c in enumerate(cols)]).astype(np.int64)
    return synth.kkt_constructed(m, n, keys, rng, name=f"{m}x{n}")


def one_workgroup():
    """The one-workgroup solver's instances with whole slices of empty rows, of empty columns, and
    with no entry at all."""
    none = synth.kkt_constructed(100, 140, np.zeros(0, np.int64), np.random.default_rng(3), name="no entries")
    for lp in (_empty_slices(200, 250, 60, 250, 1), _empty_slices(250, 200, 250, 60, 2), _empty_slices(500, 500, 100, 90, 3),
               _empty_slices(900, 1500, 100, 200, 4), none):
        for method in (0, 1):
            for prec in (0, 1):
                with lpg.Solver(lp, eps_rel=0.0, max_iters=130, spmv_layout=1, method=method, precision=prec) as s:
                    sol = s.solve()
                    assert sol.info.solve_path == 1
                    yield f"{lp.name} {method} {prec}", np.concatenate((sol.x, sol.y, sol.z))


def two_phase_products():
    """The two-phase kernels: few entries per column block, long rows in shared tiles, rows longer
    than a tile, empty rows, a last block of one column."""
    for name in ("wide", "large", "edge"):
        lp = two_phase._lp(*two_phase.CASES[name], 5)
        for prec in (0, 1):
            with lpg.Solver(lp, eps_rel=0.0, max_iters=70, method=1, precision=prec) as s:
                sol = s.solve()
                yield f"{name} {prec}", np.concatenate((sol.x, sol.y, sol.z))


def row_tiles():
    """Row tiles of one LP's own launches in both layouts, plain and non-temporal loads, rows that a
    workgroup reduces; and the batches' launches side by side."""
    rng = np.random.default_rng(8)
    keys = lambda m, n, row: np.unique(np.repeat(np.arange(m, dtype=np.int64) * n, row)  # noqa: E731
                                       + rng.integers(0, n, size=m * row))
    lps = [synth.kkt_constructed(m, n, keys(m, n, row), rng, name=f"{m}x{n}")
           for m, n, row in ((9000, 13000, 11), (900, 6000, 400), (300, 9000, 1300))]
    for lp in lps:
        for layout in (0, 1):
            for prec in (0, 1):
                with lpg.Solver(lp, eps_rel=0.0, max_iters=70, spmv_layout=layout, precision=prec, small_lp_lds=0) as s:
                    sol = s.solve()
                    yield f"{lp.name} {layout} {prec}", np.concatenate((sol.x, sol.y, sol.z))
    lps += [synth.cfg0(0), _empty_slices(300, 480, 300, 480, 1), _empty_slices(700, 1400, 700, 1400, 2),
            synth.kkt_constructed(80, 300, np.unique(np.concatenate((np.arange(140), keys(80, 300, 3)))), rng)]
    solvers = [lpg.Solver(lp, spmv_layout=1, method=1) for lp in lps]
    try:
        o = lpg.make_options(eps_rel=0.0, max_iters=70, method=1)
        lpg.lp_solve_batch_static([s.h for s in solvers], o)
        for i, s in enumerate(solvers):
            yield f"static {i}", s.iterates()[2]
    finally:
        for s in solvers:
            s.close()


SETS = {"one_workgroup": one_workgroup, "two_phase_products": two_phase_products, "row_tiles": row_tiles}

if __name__ == "__main__":
    res = dict(SETS[sys.argv[1]]())
    word, checked = lpg.lp_check_word(0)
    np.savez(sys.argv[2], word=word, checked=int(checked), **res)
    print(f"{sys.argv[1]}: {len(res)} solves, checked build {checked}, check word {word}", flush=True)
