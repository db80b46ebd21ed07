"""What a server counts for a request: no more than the arrays of the solve and of its set-up took
before the one-workgroup solver's matrices, the tile records and the two-phase layout existed. A
server iterates with row tiles; what else its set-up uses must not keep requests out."""
import numpy as np
import pytest

import paper_2604_23951_amd as lpg
import synth

pytestmark = pytest.mark.gpu


def _lps():
    rng = np.random.default_rng(3)
    rows = lambda m, n, lo, hi: np.unique(np.concatenate(  # noqa: E731
        [i * np.int64(n) + rng.integers(0, n, size=k) for i, k in enumerate(rng.integers(lo, hi, size=m))]))
    out = {"cfg0": synth.cfg0(0), "transport": synth.transportation(300, rng)}
    for name, m, n, lo, hi in (("one launch", 3000, 4500, 3, 21), ("sliced, not one launch", 4500, 6700, 3, 21),
                               ("neither", 20000, 30000, 3, 21), ("many rows", 30000, 9000, 0, 3)):
        out[name] = synth.kkt_constructed(m, n, rows(m, n, lo, hi), rng, name=name)
    return out


# layouts 0 and 1, each in FP64 and in the FP32 form
BYTES = {
    "cfg0": (709632, 756480, 654848, 688384),
    "transport": (723968, 771328, 683008, 720640),
    "one launch": (3664640, 4441856, 2541312, 3041536),
    "sliced, not one launch": (5201152, 6357760, 3532288, 4277248),
    "neither": (21319936, 26474752, 13948672, 17266944),
    "many rows": (7797504, 9490944, 6824448, 8277760),
}


@pytest.mark.parametrize("name", ["cfg0", "transport", "one launch", "sliced, not one launch", "neither", "many rows"])
def test_footprint(name):
    lp = _lps()[name]
    for i, (layout, precision) in enumerate(((0, 0), (0, 1), (1, 0), (1, 1))):
        opts = dict(spmv_layout=layout, precision=precision, method=1, eps_rel=0.0, max_iters=64)
        print(name, layout, precision, flush=True)
        with lpg.Solver(lp, small_lp_lds=0, **opts) as s:
            solo = s.solve()
        with lpg.Solver(lp, deferred=1, **opts) as t:
            with lpg.Server(BYTES[name][i], 4, **opts) as srv:  # a budget that just fitted is enough
                tickets = [srv.submit(t) for _ in range(3)]
                srv.wait(60.0)
                sols = [srv.result(k) for k in tickets]
                assert 0 < srv.stats()["peak_bytes"] <= BYTES[name][i]
        for s in sols:
            assert s.info.sigma_max == solo.info.sigma_max
            if layout == 1:
                np.testing.assert_array_equal(s.x, solo.x)
                np.testing.assert_array_equal(s.y, solo.y)
