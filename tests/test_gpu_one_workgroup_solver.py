"""The one-workgroup solver of the batched solves (every instance: 256, 512 and 1024 threads,
operands in registers or in global memory, matrices in LDS, partly staged or from the L2)
against the kernel-per-phase loop with row tiles. Both add the products of a row in CSR order
and run the same updates, so the iterates are equal bit for bit; up to 1024 rows and columns
the evaluations sum in the same order as well, so whole runs with restarts are."""
import numpy as np
import pytest

import oracle
import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu

# rows, columns, entries per row: the edges of the instances' ranges and of a 64-row slice,
# odd and even row lengths, more rows than columns
SHAPES = [(1, 1, 1), (1, 5, 5), (63, 64, 3), (64, 65, 4), (65, 256, 17), (256, 255, 9), (257, 256, 2), (200, 512, 20),
          (512, 511, 3), (513, 512, 5), (330, 660, 33), (1024, 1000, 6), (1000, 24, 7)]
WIDE = [(1024, 2048, 8), (1025, 2048, 3), (500, 2049, 40), (2048, 4096, 4), (2049, 4096, 3), (3000, 9000, 5),
        (5120, 10240, 2), (5121, 10240, 2), (6000, 1500, 3)]


def _lp(m, n, row, seed=0):
    """Row lengths from 0 to `row`, one of them exactly `row`; every column bounded."""
    rng = np.random.default_rng([m, n, row, seed])
    length = rng.integers(0, row + 1, size=m)
    length[rng.integers(0, m)] = row
    cols = [np.sort(rng.choice(n, size=min(k, n), replace=False)) for k in length]
    keys = np.concatenate([i * n + c for i, c in enumerate(cols)]).astype(np.int64)
    return synth.kkt_constructed(m, n, keys, rng, free_frac=0.1, eq_frac=0.4, two_sided_frac=0.2, name=f"{m}x{n}")


def _run(lp, iters, batch, budget=112 * 1024, **opts):
    with lpg.Solver(lp, spmv_layout=1, eps_rel=0.0, max_iters=iters, small_lp_lds=budget if batch else 0, **opts) as s:
        if batch:
            o = {k: v for k, v in opts.items() if k not in ("x0", "y0", "precision")}
            sol = lpg.solve_batch([s], eps_rel=0.0, max_iters=iters, small_lp_lds=budget, batch_split_nnz=1 << 40, **o)[0]
        else:
            sol = s.solve()
            assert sol.info.solve_path == 0
        return s.iterates(), sol


def _equal(a, b, name):
    for u, v in zip(a[0], b[0]):
        np.testing.assert_array_equal(u, v, err_msg=name)
    np.testing.assert_array_equal(a[1].x, b[1].x, err_msg=name)
    np.testing.assert_array_equal(a[1].y, b[1].y, err_msg=name)
    np.testing.assert_array_equal(a[1].z, b[1].z, err_msg=name)
    assert (a[1].status, a[1].info.iterations, a[1].info.restarts) == (b[1].status, b[1].info.iterations, b[1].info.restarts)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("method", [0, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}r{s[2]}")
def test_runs_equal_the_kernel_loop(shape, method, precision):
    lp = _lp(*shape)
    print(shape, method, precision, flush=True)
    for iters in (1, 200):
        want = _run(lp, iters, False, method=method, precision=precision)
        for budget in (112 * 1024, 20 * 1024, 0):
            _equal(_run(lp, iters, True, budget, method=method, precision=precision), want, f"{iters} {budget}")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("method", [0, 1])
@pytest.mark.parametrize("shape", WIDE, ids=lambda s: f"{s[0]}x{s[1]}r{s[2]}")
def test_wide_iterates_equal_the_kernel_loop(shape, method, precision):
    """Up to the first evaluation: beyond 1024 rows or columns its sums are blocked differently."""
    lp = _lp(*shape)
    print(shape, method, precision, flush=True)
    want = _run(lp, 64, False, method=method, precision=precision, eval_every=64)
    for budget in (112 * 1024, 0):
        got = _run(lp, 64, True, budget, method=method, precision=precision, eval_every=64)
        for u, v in zip(got[0], want[0]):
            np.testing.assert_array_equal(u, v, err_msg=str(budget))


@pytest.mark.parametrize("eval_every", [1, 63, 65, 200])
def test_periods_longer_and_shorter_than_the_weight_table(eval_every):
    lp = _lp(130, 300, 6)
    for precision in (0, 1):
        want = _run(lp, 333, False, method=1, precision=precision, eval_every=eval_every)
        _equal(_run(lp, 333, True, method=1, precision=precision, eval_every=eval_every), want, str(eval_every))


def test_long_rows_keep_the_row_tiles():
    """A row longer than one thread sums: the LP is solved over row tiles, with the same iterates."""
    lp = _lp(90, 400, 129)
    want = _run(lp, 200, False, method=1)
    _equal(_run(lp, 200, True, method=1), want, "129 entries")


def test_single_solve_beyond_one_reduction_block():
    """lp_solve on one workgroup of an LP with more than 1024 columns that the row tiles staged in
    LDS do not hold keeps the reduction blocks of the kernel loop: whole runs are equal."""
    lp = synth.transportation(601, np.random.default_rng(8))
    out = []
    for budget in (112 * 1024, 0):
        with lpg.Solver(lp, spmv_layout=1, method=1, eps_rel=0.0, max_iters=700, small_lp_lds=budget) as s:
            sol = s.solve(with_trace=True)
            assert sol.info.solve_path == (1 if budget else 0)
            out.append((s.iterates(), sol))
    _equal(out[0], out[1], "601 rows")
    np.testing.assert_array_equal(out[0][1].trace, out[1][1].trace)


@pytest.mark.parametrize("method", [0, 1])
def test_time_limited_objectives_are_the_plain_sums(oracle_lib, method):
    """A time-limited lp_solve returns the objective sums in index order: those of the oracle's
    evaluation of the returned point, bit for bit."""
    lp = synth.cfg0(0)
    for limit in (1e-7, 0.02):
        with lpg.Solver(lp, method=method, eps_rel=0.0, max_iters=10**7, time_limit_s=limit) as s:
            sol = s.solve()
        assert sol.status == "time_limit" and sol.info.solve_path == 1
        chk = oracle.kkt(lp, sol.x, sol.y)
        assert (sol.info.primal_obj, sol.info.dual_obj) == (chk["pobj"], chk["dobj"])


@pytest.mark.parametrize("shape", [s for s in SHAPES + WIDE if s[1] >= 129] + [(4000, 6000, 20)], ids=lambda s: f"{s[0]}x{s[1]}r{s[2]}")
def test_norm_estimate_equals_the_launch_per_step_iteration(shape):
    """||A~|| from one launch (every row at most 128 entries) against the same LP with one more row
    of 129 explicit zeros, which keeps the launches per step: the zeros change no sum."""
    lp = _lp(*shape)
    rows = np.repeat(np.arange(lp.m), np.diff(lp.row_ptr))
    keys = np.concatenate([rows.astype(np.int64) * lp.n + lp.col_idx, lp.m * np.int64(lp.n) + np.arange(129)])
    rp, ci, v = synth.csr_from_keys(keys, lp.m + 1, lp.n, np.concatenate([lp.vals, np.zeros(129)]))
    inf = np.inf
    big = synth.LP(lp.m + 1, lp.n, rp, ci, v, lp.c, np.append(lp.b_lo, -inf), np.append(lp.b_hi, inf), lp.x_lo, lp.x_hi)
    sigma = []
    for p in (lp, big):
        with lpg.Solver(p, spmv_layout=1, max_iters=0) as s:
            sigma.append(s.solve().info.sigma_max)
    if (max(lp.m, lp.n) + 1023) // 1024 == (max(lp.m + 1, lp.n) + 1023) // 1024:
        assert sigma[0] == sigma[1]
    else:
        assert abs(sigma[0] - sigma[1]) <= 1e-12 * sigma[1]


@pytest.mark.parametrize("precision", [0, 1])
def test_the_latest_point_is_returned(precision):
    """Points written to host memory by the solve's kernel (one workgroup, batches) and copied
    from the device (kernel loop, polishing, pauses) replace each other."""
    lp = _lp(130, 300, 6)
    opts = dict(method=1, precision=precision, eps_rel=0.0)
    ref = {k: _run(lp, k, False, method=1, precision=precision)[1].x for k in (64, 128, 192)}
    with lpg.Solver(lp, spmv_layout=1, max_iters=64, **opts) as s:
        np.testing.assert_array_equal(s.solve().x, ref[64])
        s.update(max_iters=1000, **{k: v for k, v in opts.items() if k != "precision"})
        np.testing.assert_array_equal(s.solve_until(128).x, ref[128])
        np.testing.assert_array_equal(lpg.solve_batch([s], max_iters=64, **opts)[0].x, ref[64])
        np.testing.assert_array_equal(lpg.solve_batch([s], max_iters=192, batch_split_nnz=0, **opts)[0].x, ref[192])
        s.update(max_iters=128, **{k: v for k, v in opts.items() if k != "precision"})
        a = s.solve()
        np.testing.assert_array_equal(a.x, ref[128])
        p = s.polish(1e-6, 200)
        again = np.empty(lp.n)
        lpg.lp_get_solution(s.h, again)
        np.testing.assert_array_equal(again, p.x)
        assert not np.array_equal(p.x, a.x)
