"""Solves run by tests/test_gpu_checked_forms.py, in that process with the plain build and in one of
its own with the bounds-checked build (LPGPU_CHECKED=1); there it writes the returned points and the
check word to the .npz file named on the command line."""
import sys

import numpy as np

import paper_2604_23951_amd as lpg
import synth


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


SETS = {"one_workgroup": one_workgroup}

if __name__ == "__main__":
    res = dict(SETS[sys.argv[1]]())
    word, checked = lpg.lp_check_word(0)
    np.savez(sys.argv[2], word=word, checked=int(checked), **res)
    print(f"{sys.argv[1]}: {len(res)} solves, checked build {checked}, check word {word}", flush=True)
