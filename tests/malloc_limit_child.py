"""Run by test_gpu_out_of_memory.py: creates and solves an LP of the two-phase layout while hipMalloc
refuses what that layout adds to its allocation (or the layout's set-up buffer)."""
import ctypes
import sys

shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.shim_limit.argtypes = [ctypes.c_size_t]

import numpy as np  # noqa: E402

import paper_2604_23951_amd as lpg  # noqa: E402
import synth  # noqa: E402

rng = np.random.default_rng(5)
m, n = 40000, 600011
lp = synth.kkt_constructed(m, n, np.unique(rng.integers(0, m, size=200000) * n + rng.integers(0, n, size=200000)), rng)


def solve(**opts):
    with lpg.Solver(lp, method=1, eps_rel=0.0, max_iters=40, **opts) as s:
        sol = s.solve()
        lay = s.layout()
        return lay["two_phase_a"], lay["device_bytes"], [sol.x, sol.y, sol.z, *s.iterates()]


tiles, full, want = solve()
none, panels, other = solve(panel_slice_bytes=(1 << 19) - 8)
assert tiles > 0 and none == 0 and full > panels, (tiles, none, full, panels)
print(full, panels, flush=True)
assert shim.shim_refused() == 0
shim.shim_limit(panels + (full - panels) // 2)
got = [solve()]
assert shim.shim_refused() == 1 and got[0][1] < full
shim.shim_limit(1 << 60)
shim.shim_refuse_call(2)  # the set-up buffer, after the handle's own memory
got.append(solve())
assert shim.shim_refused() == 2 and got[1][1] == full
for tiles, _, point in got:
    assert tiles == 0
    for a, b in zip(point, want):
        np.testing.assert_array_equal(a, b)
shim.shim_limit(1 << 20)
try:
    solve()
    raise SystemExit("an allocation that fails without the layout too is an error")
except lpg.LpError as e:
    print(e, flush=True)
print("ok")
