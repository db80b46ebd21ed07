"""Run by test_gpu_out_of_memory.py: solves a small LP, alone and in a batch, while hipHostMalloc
refuses the pinned memory for its point."""
import ctypes
import sys

shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.shim_host_limit.argtypes = [ctypes.c_size_t]

import numpy as np  # noqa: E402

import paper_2604_23951_amd as lpg  # noqa: E402
import synth  # noqa: E402


def solve():
    with lpg.Solver(synth.cfg0(0), spmv_layout=1, eps_rel=0.0, max_iters=200) as s:
        sols = [s.solve(), lpg.solve_batch([s], eps_rel=0.0, max_iters=128)[0]]
        assert sols[0].info.solve_path == 1
        return [v for q in sols for v in (q.x, q.y, q.z, np.array([q.info.rel_kkt, q.info.primal_obj]))]


want = solve()
assert shim.shim_refused() == 0
shim.shim_host_limit(512)  # the scalar state alone
got = solve()
assert shim.shim_refused() >= 1
for a, b in zip(got, want):
    np.testing.assert_array_equal(a, b)
print("ok")
