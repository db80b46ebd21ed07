"""Performance cases of the LP solver: what is timed, on which inputs, and the value each pass should give.

Every case is one call (or one round of calls) that a program using the solver makes, through
the Python entry points of paper_2604_23951_amd. A solve runs a fixed number of iterations
(eps_rel = 0 with max_iters set), the way a solve to a tolerance spends its time, so that two
builds do the same work. Shapes follow the workloads of the benchmark and the tests:

  sparse     n about 2m, Bernoulli pattern of a given density (the small LP and the batch)
  rows       n about 1.5m, 3 to 20 entries per row (the serving pool)
  power      n about 2m, about 12 entries per row, power-law column degrees (the large LP)
  transport  supply / demand rows, two entries per column (the other half of the batch)
  planted    `sparse` with fixed columns, singleton and redundant rows (presolve)

Kinds of call:

  solve      Solver.solve() on a handle set up before
  batch      solve_batch() over `count` handles, rows log-uniform in [m_lo, m]
  static     the same through lp_solve_batch_static (no device allocation in the call)
  serve      `count` requests put through a running Server: set-up, solve and result of each
  presolved  solve_presolved(): presolve, set-up, solve and postsolve of a new LP
"""
import math

import numpy as np
import torch

import paper_2604_23951_amd as lpg

SEED_ROOT = 260423951
HALPERN = {"method": 1}
INF = math.inf


def listed():
    return [
        # the smallest call: a toy LP with every option at its default (averaged form, FP64)
        dict(name="solve_tiny_default", kind="solve", recipe="sparse", m=50, n=100, density=0.05, method=0, fp32=False,
             layout=0, iters=2048),
        # the small LP of the benchmark with the latency preset
        dict(name="solve_small", kind="solve", recipe="sparse", m=200, n=400, density=0.02, method=1, fp32=False,
             layout=1, iters=4096),
        # a few hundred rows, too large for one workgroup's LDS
        dict(name="solve_transport", kind="solve", recipe="transport", m=601, n=1202, method=1, fp32=False, layout=0,
             iters=1024),
        # a mid-sized LP of the serving pool on its own
        dict(name="solve_mid_fp32", kind="solve", recipe="rows", m=20011, n=30017, method=1, fp32=True, layout=1,
             iters=768),
        # the densest LP of the batch recipe's size range, every option at its default
        dict(name="solve_dense_default", kind="solve", recipe="sparse", m=4999, n=9998, density=0.02, method=0,
             fp32=False, layout=0, iters=384),
        # the headline LP: m = 1e6, n = 2e6, 1.2e7 nonzeros, large-LP preset
        dict(name="solve_large", kind="solve", recipe="power", m=1000000, n=2000000, method=1, fp32=False, layout=0,
             iters=256),
        # a large LP in the FP32 storage form, ragged sizes
        dict(name="solve_large_fp32", kind="solve", recipe="power", m=600011, n=1200007, method=1, fp32=True, layout=0,
             iters=256),
        # an uneven batch of the batched workload: both recipes, 50 to 5000 rows
        dict(name="batch_mixed", kind="batch", recipe="mixed", m_lo=50, m=5000, count=96, method=1, fp32=True,
             layout=1, iters=512),
        # a batch of small LPs in FP64
        dict(name="batch_small_fp64", kind="batch", recipe="mixed", m_lo=50, m=330, count=128, method=1, fp32=False,
             layout=1, iters=1024),
        # the allocation-free batch
        dict(name="static_batch", kind="static", recipe="mixed", m_lo=50, m=900, count=64, method=1, fp32=True,
             layout=1, iters=512),
        # requests of the serving pool put through a server
        dict(name="serve", kind="serve", recipe="rows", m_lo=100, m=20000, count=32, method=1, fp32=True, layout=1,
             iters=512),
        # a new LP solved from scratch: presolve, set-up, solve, postsolve
        dict(name="presolved", kind="presolved", recipe="planted", m=3001, n=6007, density=0.002, method=1, fp32=False,
             layout=0, iters=1024),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["batch", "batch", "static", "serve", "presolved"])
    c = dict(kind=kind, method=rng.choice([0, 1, 1]), fp32=rng.choice([False, True]), layout=rng.choice([0, 1]))
    if kind == "solve":
        c["recipe"] = rng.choice(["sparse", "transport", "rows", "rows", "power"])
        if c["recipe"] == "power":
            c["m"] = _log_uniform(rng, 20000, 900000)
            c["n"] = 2 * c["m"] + rng.randrange(-7, 8)
        elif c["recipe"] == "rows":
            c["m"] = _log_uniform(rng, 100, 200000)
            c["n"] = (3 * c["m"]) // 2 + rng.randrange(0, 9)
        else:
            c["m"] = _log_uniform(rng, 50, 5000)
            c["n"] = 2 * c["m"]
            if c["recipe"] == "sparse":
                c["density"] = round(rng.uniform(0.005, 0.05), 4)
        c["iters"] = int(min(4096, max(128, 3.0e9 / (12.0 * _nnz(c) + 3.0e6)))) // 64 * 64 + rng.choice([0, 0, 17])
    elif kind in ("batch", "static"):
        small = kind == "static" or rng.random() < 0.5
        c.update(recipe="mixed", m_lo=50, m=_log_uniform(rng, 100, 900) if small else rng.randrange(1500, 5001),
                 count=rng.randrange(20, 97), iters=rng.choice([256, 384, 512]), layout=1)
    elif kind == "serve":
        c.update(recipe="rows", m_lo=100, m=_log_uniform(rng, 2000, 20000), count=rng.randrange(8, 33), iters=320, layout=1)
    else:
        m = rng.randrange(500, 4001)
        c.update(recipe="planted", m=m, n=2 * m + rng.randrange(0, 9), density=round(rng.uniform(0.001, 0.004), 4), iters=512)
    return c


# ------------------------------------------------------------------------------ inputs

class Problem:
    """An LP with the fields the solver's binding reads."""

    def __init__(self, m, n, keys, vals):
        self.m, self.n, self.c0 = m, n, 0.0
        rows = keys // n
        self.rows = rows.astype(np.int32)
        self.col_idx = (keys - rows * n).astype(np.int32)
        self.vals = vals
        self.row_ptr = np.zeros(m + 1, np.int32)
        np.cumsum(np.bincount(rows, minlength=m), out=self.row_ptr[1:])

    def product(self, x):
        return np.bincount(self.rows, weights=self.vals * x[self.col_idx], minlength=self.m)

    def transposed(self, y):
        return np.bincount(self.col_idx, weights=self.vals * y[self.rows], minlength=self.n)


def _unique(keys):
    keys.sort()
    return keys[np.concatenate(([True], keys[1:] != keys[:-1]))]


def _pattern(recipe, m, n, density, rng):
    """Sorted keys row * n + column; every row holds an entry."""
    base = np.arange(m, dtype=np.int64) * n
    if recipe == "rows":
        k = rng.integers(3, 21, size=m)
        return _unique(np.repeat(base, k) + rng.integers(0, n, size=int(k.sum())))
    if recipe == "power":  # column degrees d^-2.2 on [1, 5000], two entries in every row, uniform ones up to 12 a row
        d = np.arange(1, min(5000, m) + 1, dtype=np.float64) ** -2.2
        deg = np.searchsorted(np.cumsum(d / d.sum()), rng.random(n)) + 1
        cols = np.repeat(np.arange(n, dtype=np.int64), deg)
        parts = [rng.integers(0, m, size=len(cols)) * n + cols]
        parts += [base + rng.integers(0, n, size=m) for _ in range(2)]
        extra = max(0, 12 * m - sum(map(len, parts)))
        parts.append(rng.integers(0, m, size=extra) * n + rng.integers(0, n, size=extra))
        return _unique(np.concatenate(parts))
    extra = rng.binomial(m * n, density)
    return _unique(np.concatenate((base + rng.integers(0, n, size=m), rng.integers(0, m * n, size=extra))))


def _transport(m, rng):
    S = m // 2
    D, n = m - S, 2 * m
    k = np.arange(max(S, D))
    need = (k % S) * D + k % D
    # every row has an edge; the other edges are distinct random pairs
    rest = _unique(rng.integers(0, S * D, size=4 * n))
    rest = rng.permutation(rest[~np.isin(rest, need)])
    pairs = rng.permutation(np.concatenate((need, rest))[:n])
    n = len(pairs)
    sup, dem = pairs // D, S + pairs % D
    col = np.arange(n)
    lp = Problem(m, n, np.sort(np.concatenate((sup * n + col, dem * n + col))), np.ones(2 * n))
    ax = lp.product(rng.random(n))
    lp.b_lo = np.where(np.arange(m) < S, -INF, ax)
    lp.b_hi = np.where(np.arange(m) < S, ax + 1.0 - rng.random(m), INF)
    lp.c = rng.uniform(1.0, 100.0, size=n)
    lp.x_lo, lp.x_hi = np.zeros(n), np.full(n, INF)
    return lp


def _problem(c, m, n, recipe, density, rng):
    """An LP with a known optimal pair (x*, y*, z*): bounds and costs follow from it."""
    if recipe == "transport":
        return _transport(m, rng)
    keys = _pattern(recipe, m, n, density, rng)
    planted = recipe == "planted"
    if planted:  # a tenth of the rows keep one entry
        single = rng.random(m) < 0.1
        rows = keys // n
        first = np.concatenate(([True], rows[1:] != rows[:-1]))
        keys = keys[first | ~single[rows]]
    lp = Problem(m, n, keys, rng.standard_normal(len(keys)))
    free = rng.random(n) < (0.2 if recipe == "power" else 0.0)
    low = ~free & (rng.random(n) < 0.5)
    x = np.where(free, rng.standard_normal(n), np.where(low, 0.0, 1.0 - rng.random(n)))
    z = np.where(low, 1.0 - rng.random(n), 0.0)
    lp.x_lo, lp.x_hi = np.where(free, -INF, 0.0), np.where(free, INF, 10.0)
    ax = lp.product(x)
    u = rng.random(m)
    two = 0.3 if recipe == "power" else 0.0
    eq, both = u < 0.5 - two / 2, (u >= 0.5 - two / 2) & (u < 0.5 + two / 2)
    slack, gap, size = rng.random(m) < 0.5, 1.0 - rng.random(m), rng.standard_normal(m)
    y = np.where(eq, size, np.where(slack, 0.0, np.abs(size)))
    if planted:  # fixed columns, and slack rows that no point within the bounds violates
        fixed = rng.random(n) < 0.1
        lp.x_lo, lp.x_hi = np.where(fixed, x, lp.x_lo), np.where(fixed, x, lp.x_hi)
        z = np.where(fixed, rng.standard_normal(n), z)
        gap = np.where(rng.random(m) < 0.4, 1000.0, gap)
    lp.b_lo = np.where(eq, ax, np.where(slack, ax - gap, ax))
    lp.b_hi = np.where(eq, ax, np.where(both, ax + gap, INF))
    lp.c = lp.transposed(y) + z
    return lp


def _problems(case, seed):
    rng = np.random.default_rng([SEED_ROOT, seed])
    if "count" not in case:
        return [_problem(case, case["m"], case["n"], case["recipe"], case.get("density", 0.0), rng)]
    out = []
    sizes = np.exp(np.linspace(math.log(case["m_lo"]), math.log(case["m"]), case["count"]))
    for i, m in enumerate(np.round(sizes).astype(int).tolist()):
        recipe = case["recipe"] if case["recipe"] != "mixed" else ("sparse", "transport")[i % 2]
        n = (3 * m) // 2 if recipe == "rows" else 2 * m
        out.append(_problem(case, m, n, recipe, 0.005 + 0.045 * ((7 * i) % 16) / 16.0, rng))
    return out


def _options(case):
    return dict(method=case["method"], precision=int(case["fp32"]), spmv_layout=case["layout"], eps_rel=0.0,
                max_iters=case["iters"])


def prepare(case, seed):
    lps, opt = _problems(case, seed), _options(case)
    st = {"kind": case["kind"], "opt": opt}
    if case["kind"] == "presolved":
        st["lp"] = lps[0]
    else:
        st["solvers"] = [lpg.Solver(lp, deferred=int(case["kind"] == "serve"), **opt) for lp in lps]
    if case["kind"] == "serve":
        st["server"] = lpg.Server(hbm_budget_bytes=32 << 30, max_slots=64, **opt)
    return st


def _outputs(sols):
    cat = (lambda k: getattr(sols[0], k)) if len(sols) == 1 else (lambda k: np.concatenate([getattr(s, k) for s in sols]))
    infos = [s.info for s in sols]
    return {"x": cat("x"), "y": cat("y"), "z": cat("z"),
            "iterations": np.array([i.iterations for i in infos]), "restarts": np.array([i.restarts for i in infos]),
            "status": np.array([i.status for i in infos]), "rel_kkt": np.array([i.rel_kkt for i in infos]),
            "objective": np.array([[i.primal_obj, i.dual_obj] for i in infos])}


def run(state):
    kind = state["kind"]
    if kind == "solve":
        return _outputs([state["solvers"][0].solve()])
    if kind == "batch":
        return _outputs(lpg.solve_batch(state["solvers"], **state["opt"]))
    if kind == "static":
        solvers = state["solvers"]
        lpg.lp_solve_batch_static([s.h for s in solvers], lpg.make_options(**state["opt"]))
        sols = []
        for s in solvers:
            x, y, z = np.empty(s.n), np.empty(s.m), np.empty(s.n)
            sols.append(lpg.Solution("", x, y, z, lpg.lp_get_solution(s.h, x, y, z)))
        return _outputs(sols)
    if kind == "serve":
        server = state["server"]
        tickets = [server.submit(s) for s in state["solvers"]]
        server.wait()
        server.poll(len(tickets))
        return _outputs([server.result(t) for t in tickets])
    r = lpg.solve_presolved(state["lp"], **state["opt"])
    return {"x": r.x, "y": r.y, "z": r.z, "reduced_iterations": np.array([r.reduced.info.iterations])}


# ------------------------------------------------------------------ what a pass needs

def _nnz(case, m=None, n=None, density=None, recipe=None):
    m, n = m or case["m"], n or case["n"]
    recipe = recipe or case["recipe"]
    if recipe == "transport":
        return 2.0 * n
    if recipe == "rows":
        return 11.5 * m
    if recipe == "power":
        return 12.0 * m
    return m + (density if density is not None else case["density"]) * m * n


def work(case):
    """Per iteration: the matrix and its transpose (value and column of every entry, row
    pointers), each vector of the two fused updates read or written once, two operations per
    entry and product; times the iterations. Every matrix is streamed once per iteration, as it
    must be where it does not fit on the chip."""
    sv = 4 if case["fp32"] else 8
    shapes = []
    if "count" in case:
        for i, m in enumerate(np.exp(np.linspace(math.log(case["m_lo"]), math.log(case["m"]), case["count"]))):
            recipe = case["recipe"] if case["recipe"] != "mixed" else ("sparse", "transport")[i % 2]
            n = (1.5 if recipe == "rows" else 2.0) * m
            shapes.append((m, n, _nnz(case, m, n, 0.005 + 0.045 * ((7 * i) % 16) / 16.0, recipe)))
    else:
        shapes.append((case["m"], case["n"], _nnz(case)))
    per_iter = sum(2 * (sv + 4) * z + 4 * (m + n + 2) + sv * (8 * n + 9 * m) for m, n, z in shapes)
    return {"bytes": case["iters"] * per_iter, "flops": case["iters"] * 4.0 * sum(z for _, _, z in shapes)}


# ------------------------------------------------------------- the same in plain torch

class _Reference:
    """The restarted PDHG iteration in 64-bit torch over all LPs of a case at once: vectors
    are concatenated, scalars are one per LP."""

    def __init__(self, lps):
        dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        t = lambda parts: torch.from_numpy(np.concatenate(parts)).to(dev)  # noqa: E731
        self.dev, self.k = dev, len(lps)
        mo = np.cumsum([0] + [lp.m for lp in lps])
        no = np.cumsum([0] + [lp.n for lp in lps])
        self.m, self.n = int(mo[-1]), int(no[-1])
        self.row = t([lp.rows.astype(np.int64) + o for lp, o in zip(lps, mo)])
        self.col = t([lp.col_idx.astype(np.int64) + o for lp, o in zip(lps, no)])
        self.a = t([lp.vals for lp in lps])
        self.rl = t([np.full(lp.m, i) for i, lp in enumerate(lps)])
        self.cl = t([np.full(lp.n, i) for i, lp in enumerate(lps)])
        self.c, self.bl, self.bu = t([lp.c for lp in lps]), t([lp.b_lo for lp in lps]), t([lp.b_hi for lp in lps])
        self.xl, self.xu = t([lp.x_lo for lp in lps]), t([lp.x_hi for lp in lps])
        self.local = t([np.arange(lp.n) for lp in lps]).cpu().numpy()
        self._scale()
        self._step()

    def A(self, x):
        return torch.zeros(self.m, dtype=torch.float64, device=self.dev).index_add_(0, self.row, self.a * x[self.col])

    def At(self, y):
        return torch.zeros(self.n, dtype=torch.float64, device=self.dev).index_add_(0, self.col, self.a * y[self.row])

    def _sum(self, v, lp):
        if self.k == 1:
            return v.sum()[None]
        return torch.zeros(self.k, dtype=torch.float64, device=self.dev).index_add_(0, lp, v)

    def rows(self, v):
        return self._sum(v, self.rl)

    def cols(self, v):
        return self._sum(v, self.cl)

    def _scale(self):
        """Ten passes by the largest entry and one by the sum, in powers of two."""
        def factor(v):
            e = torch.frexp(v)[1].to(torch.float64)
            return torch.where(v > 0, torch.pow(2.0, -torch.floor(e / 2)), torch.ones_like(v))

        z = lambda k: torch.zeros(k, dtype=torch.float64, device=self.dev)  # noqa: E731
        self.R, self.C = z(self.m) + 1, z(self.n) + 1
        for p in range(11):
            b = self.a.abs()
            if p < 10:
                r, c = z(self.m).scatter_reduce_(0, self.row, b, "amax"), z(self.n).scatter_reduce_(0, self.col, b, "amax")
            else:
                r, c = z(self.m).index_add_(0, self.row, b), z(self.n).index_add_(0, self.col, b)
            r, c = factor(r), factor(c)
            self.a = self.a * r[self.row] * c[self.col]
            self.R, self.C = self.R * r, self.C * c
        q = lambda lo, hi: torch.maximum(torch.where(lo.isfinite(), lo.abs(), 0.0), torch.where(hi.isfinite(), hi.abs(), 0.0))  # noqa: E731
        self.cnorm, self.qnorm = self.cols(self.c ** 2).sqrt(), self.rows(q(self.bl, self.bu) ** 2).sqrt()
        self.c, self.bl, self.bu = self.c * self.C, self.bl * self.R, self.bu * self.R
        self.xl, self.xu = self.xl / self.C, self.xu / self.C
        cs, qs = self.cols(self.c ** 2).sqrt(), self.rows(q(self.bl, self.bu) ** 2).sqrt()
        self.omega = torch.where((cs > 1e-10) & (qs > 1e-10), cs / qs, torch.ones_like(cs))

    def _step(self):
        """0.998 / ||A||: the power iteration from the solver's start vector."""
        with np.errstate(over="ignore"):
            s = np.uint64(0x5EED0C0FFEE) + (self.local.astype(np.uint64) + np.uint64(1)) * np.uint64(0x9E3779B97F4A7C15)
            s = (s ^ (s >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            s = (s ^ (s >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            s ^= s >> np.uint64(31)
        v = torch.from_numpy((s >> np.uint64(11)).astype(np.float64) / 2.0 ** 53 - 0.5).to(self.dev)
        v = v / self.cols(v * v).sqrt()[self.cl]
        sigma = torch.zeros(self.k, dtype=torch.float64, device=self.dev)
        live = torch.ones_like(sigma, dtype=torch.bool)
        for _ in range(25):
            for _ in range(200):
                u = self.A(v)
                w = self.At(u)
                before, now = sigma, self.rows(u * u).sqrt()
                v = torch.where(live[self.cl], w / self.cols(w * w).sqrt()[self.cl], v)
                sigma = torch.where(live, now, sigma)
            live = live & (sigma - before > 1e-8 * sigma)
            if not bool(live.any()):
                break
        self.eta = 0.998 / sigma

    def kkt(self, x, y, ax, aty, xan, yan):
        rs = ax - torch.minimum(torch.maximum(ax, self.bl), self.bu)
        lam = self.c - aty
        flo, fhi = self.xl.isfinite(), self.xu.isfinite()
        z = torch.where(flo & fhi, lam, torch.where(flo, lam.clamp(min=0), torch.where(fhi, lam.clamp(max=0), 0.0)))
        yo, zero = y * self.R, torch.zeros((), dtype=torch.float64, device=self.dev)
        vs = torch.where(self.bl == -INF, y.clamp(min=0), zero) - torch.where(self.bu == INF, y.clamp(max=0), zero)
        dobj = self.rows(torch.where((yo > 0) & self.bl.isfinite(), self.bl * y, zero) + torch.where((yo < 0) & self.bu.isfinite(), self.bu * y, zero))
        dobj = dobj + self.cols(torch.where(z > 0, self.xl * z, zero) + torch.where(z < 0, self.xu * z, zero))
        pobj = self.cols(self.c * x)
        rd = lam - z
        k = dict(p=pobj, d=dobj, rp=self.rows(rs ** 2), rd=self.rows(vs ** 2) + self.cols(rd ** 2),
                 dx=self.cols((x - xan) ** 2).sqrt(), dy=self.rows((y - yan) ** 2).sqrt(), z=z / self.C)
        rel_p = self.rows((rs / self.R) ** 2).sqrt() / (1 + self.qnorm)
        rel_d = (self.rows((vs * self.R) ** 2) + self.cols((rd / self.C) ** 2)).sqrt() / (1 + self.cnorm)
        gap = (pobj - dobj).abs() / (1 + pobj.abs() + dobj.abs())
        k["e"] = torch.maximum(torch.maximum(rel_p, rel_d), gap)
        return k

    def weighted(self, k, om):
        return (om ** 2 * k["rp"] + k["rd"] / om ** 2 + (k["p"] - k["d"]) ** 2).sqrt()

    def solve(self, halpern, iters, every=64):
        x = torch.minimum(torch.maximum(torch.zeros_like(self.c), self.xl), self.xu)
        y = torch.zeros_like(self.bl)
        xa, ya, xan, yan, ax = x, y, x, y, self.A(x)
        axan, axa, om = ax, ax, self.omega
        anchor = self.weighted(self.kkt(x, y, ax, self.At(y), xan, yan), om)
        prev = torch.full_like(om, INF)
        k, t = 0, torch.zeros_like(om)
        restarts = torch.zeros_like(om)
        while True:
            tau, sig = (self.eta / om)[self.cl], (self.eta * om)[self.rl]
            steps = min(every, iters - k)
            for i in range(steps):
                xp = x - tau * (self.c - self.At(y))
                xp = torch.minimum(torch.maximum(xp, self.xl), self.xu)
                s = self.A(xp)
                v = y - sig * (2 * s - ax)
                yp = (v + sig * self.bl).clamp(min=0) + (v + sig * self.bu).clamp(max=0)
                if halpern:
                    w = (t + i + 1) / (t + i + 2)
                    wc, wr = w[self.cl], w[self.rl]
                    x, y = wc * (2 * xp - x) + (1 - wc) * xan, wr * (2 * yp - y) + (1 - wr) * yan
                    ax = wr * (2 * s - ax) + (1 - wr) * axan
                    xa, ya, axa = xp, yp, s
                else:
                    w = 1 / (t + i + 1)
                    x, y, ax = xp, yp, s
                    xa, ya = xa + w[self.cl] * (x - xa), ya + w[self.rl] * (y - ya)
                    if k + i == 0 or bool((t + i == 0).any()):
                        first = t + i == 0
                        xa, ya = torch.where(first[self.cl], x, xa), torch.where(first[self.rl], y, ya)
            k, t = k + steps, t + steps
            if not halpern:
                axa = self.A(xa)
            avg = self.kkt(xa, ya, axa, self.At(ya), xan, yan)
            cur = avg if halpern else self.kkt(x, y, ax, self.At(y), xan, yan)
            if k >= iters:
                break
            kc, ka = self.weighted(cur, om), self.weighted(avg, om)
            use = torch.ones_like(om, dtype=torch.bool) if halpern else ka < kc
            cand = torch.where(use, ka, kc)
            again = (cand <= 0.2 * anchor) | ((cand <= 0.8 * anchor) & (cand > prev)) | (t >= 0.36 * k)
            pick = {q: torch.where(use, avg[q], cur[q]) for q in ("rp", "rd", "p", "d", "dx", "dy")}
            new = om
            for _ in range(2 if halpern else 1):
                new = (new * pick["dy"] / pick["dx"]).sqrt()
            om = torch.where(again & (pick["dx"] > 1e-10) & (pick["dy"] > 1e-10), new, om)
            anchor = torch.where(again, self.weighted(pick, om), anchor)
            prev = torch.where(again, torch.full_like(prev, INF), cand)
            t, restarts = torch.where(again, torch.zeros_like(t), t), restarts + again
            ac, ar, uc, ur = again[self.cl], again[self.rl], use[self.cl], use[self.rl]
            cx, cy, cax = torch.where(uc, xa, x), torch.where(ur, ya, y), torch.where(ur, axa, ax)
            x, xa, xan = torch.where(ac, cx, x), torch.where(ac, cx, xa), torch.where(ac, cx, xan)
            y, ya, yan = torch.where(ar, cy, y), torch.where(ar, cy, ya), torch.where(ar, cy, yan)
            ax, axan = torch.where(ar, cax, ax), torch.where(ar, cax, axan)
        use = torch.ones_like(om, dtype=torch.bool) if halpern else avg["e"] < cur["e"]
        uc, ur = use[self.cl], use[self.rl]
        return {"x": torch.where(uc, xa, x) * self.C, "y": torch.where(ur, ya, y) * self.R,
                "z": torch.where(uc, avg["z"], cur["z"]), "rel_kkt": torch.where(use, avg["e"], cur["e"]),
                "objective": torch.stack([torch.where(use, avg[q], cur[q]) for q in ("p", "d")], 1),
                "iterations": None, "restarts": None, "status": None}


def exact(case, seed):
    if case["kind"] == "presolved":  # which reductions apply is the presolver's own choice
        return None
    return _Reference(_problems(case, seed)).solve(case["method"] == 1, case["iters"])
