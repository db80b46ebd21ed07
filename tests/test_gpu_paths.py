"""Which kernels run an LP (lp_get_layout): the comparisons of one path with another say nothing
where both sides take the same one."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth
import test_gpu_two_phase as two_phase

pytestmark = pytest.mark.gpu

# (A, A^T) in two phases, per precision
EXPECT = {"wide": ((True, False), (True, False)), "large": ((True, True), (True, True)),
          "edge": ((True, False), (False, False))}


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", list(two_phase.CASES))
def test_two_phase_cases_take_the_path(name, precision):
    """The LPs of test_gpu_two_phase.py: their default runs are in two phases (where the rule says
    so), the runs they are compared with are not."""
    lp = two_phase._lp(*two_phase.CASES[name], 5)
    print(name, precision, flush=True)
    for opts, want in (({}, EXPECT[name][precision]), (dict(panel_slice_bytes=(1 << 19) - 8), (False, False))):
        with lpg.Solver(lp, precision=precision, max_iters=64, eps_rel=0.0, **opts) as s:
            s.solve()
            lay = s.layout()
        assert (lay["two_phase_a"] > 0, lay["two_phase_at"] > 0) == want
        assert lay["last_solver"] == 0 and lay["layout"] == 0


@pytest.mark.parametrize("precision", [0, 1])
def test_two_phase_with_other_options(precision):
    """Residual restarts, certificates and a pause in the two-phase products: as in the panels."""
    lp = two_phase._lp(*two_phase.CASES["large"], 6)
    out = []
    for opts in ({}, dict(panel_slice_bytes=(1 << 19) - 8)):
        print(precision, opts, flush=True)
        with lpg.Solver(lp, method=1, precision=precision, restart_metric=1, eps_infeas=1e-6, eps_rel=0.0, max_iters=150,
                        eval_every=25, **opts) as s:
            assert (s.layout()["two_phase_a"] > 0) == (not opts)
            mid = s.solve_until(50)
            end = s.resume()
            out.append([mid.x, mid.y, end.x, end.y, end.z, *s.iterates(), np.array([end.info.rel_kkt, end.info.restarts])])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


def test_two_phase_beyond_the_infinity_cache():
    """More than 192 MB an iteration: the instances with non-temporal loads."""
    lp = two_phase._lp(400001, 800009, 6700000, [300, 5000], [4999, 16000], 7)
    assert lp.nnz * 32 > 192 << 20
    out = []
    for opts in ({}, dict(panel_slice_bytes=(1 << 19) - 8)):
        print(opts, flush=True)
        with lpg.Solver(lp, method=1, eps_rel=0.0, max_iters=40, **opts) as s:
            sol = s.solve()
            assert (s.layout()["two_phase_a"] > 0, s.layout()["two_phase_at"] > 0) == ((not opts,) * 2)
            out.append([sol.x, sol.y, sol.z, *s.iterates()])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


def test_solvers_of_a_batch_are_reported():
    rng = np.random.default_rng(2)
    wide = np.concatenate([np.arange(129), 400 + np.sort(rng.choice(400, 3, replace=False))]).astype(np.int64)
    lps = [synth.cfg0(0), synth.kkt_constructed(60, 400, np.unique(np.concatenate(
        [wide, np.arange(60) * 400 + 7])), rng, name="one long row"), synth.cfg4_lp(4, m_hi=600)]
    solvers = [lpg.Solver(lp, spmv_layout=1, max_iters=64, eps_rel=0.0) for lp in lps]
    try:
        assert all(s.layout()["last_solver"] == -1 for s in solvers)
        lpg.solve_batch(solvers, max_iters=64, eps_rel=0.0)
        assert [s.layout()["last_solver"] for s in solvers[:2]] == [1, 2]
        lpg.solve_batch(solvers, max_iters=64, eps_rel=0.0, batch_split_nnz=0)
        assert [s.layout()["last_solver"] for s in solvers] == [4, 4, 4]
        lpg.lp_solve_batch_static([s.h for s in solvers], lpg.make_options(max_iters=64, eps_rel=0.0))
        assert [s.layout()["last_solver"] for s in solvers[:2]] == [1, 2]
        assert [s.solve().info.solve_path for s in solvers[:2]] == [1, 1]
        assert [s.layout()["last_solver"] for s in solvers[:2]] == [1, 2]
        solvers[0].solve_until(64)
        assert solvers[0].layout()["last_solver"] == 0
    finally:
        for s in solvers:
            s.close()
