"""Timed cases of the library's public entry points.

Each case is one call (or the short sequence of calls) that a program makes
in its inner loop, on the two synthetic sets the tests and the benchmark use:

  one    50 x knots x 30 Q knots in one sub-grid, 11 stored flavours
  three  196 x knots x 3 sub-grids of 17 Q knots (flavour thresholds), 13
         stored flavours

Grid values, query points, weights and tables are drawn from the seed.
"""
import math

import numpy as np
import torch

from paper_2009_06635_amd import pdfmi

DEV = "cuda"
PIDS = {"one": [-5, -4, -3, -2, -1, 21, 1, 2, 3, 4, 5],
        "three": [-6, -5, -4, -3, -2, -1, 21, 1, 2, 3, 4, 5, 6]}
ALL13 = ",".join(str(p) for p in PIDS["three"])
X_MIN = {"one": 1e-6, "three": 1e-9}
Q_EDGES = {"one": (1.65, 1e4), "three": (1.0, 1.51, 4.92, 1e5)}
N_X = {"one": 50, "three": 196}
N_Q = {"one": 30, "three": 17}
FK_NX, FK_Q = 2415, 1.65   # x points and scale of a multi-member evaluation for kernel-table predictions
SUR_SHAPES = ((64, 2), (64,), (64, 64), (64,), (64, 64), (64,), (16, 64), (16,))


def listed():
    return [
        # a handful of points inside a host loop: latency of one call
        {"name": "xfxq2_1e3", "op": "xfxq2", "grid": "one", "n": 1000, "pids": "all", "f32": False, "alphas": False,
         "outside": 0.0},
        # an ordinary call of a few events' worth of points
        {"name": "xfxq2_1e5", "op": "xfxq2", "grid": "one", "n": 100_000, "pids": "all", "f32": False,
         "alphas": False, "outside": 0.0},
        # the benchmark's headline: every flavour and alpha_s at 1e7 points, 1 % outside the grid
        {"name": "xfxq2_alphas_1e7", "op": "xfxq2", "grid": "three", "n": 10_000_000, "pids": "all", "f32": False,
         "alphas": True, "outside": 0.01},
        # an integrand that is content with FP32 arithmetic, on a ragged count
        {"name": "xfxq2_alphas_f32", "op": "xfxq2", "grid": "three", "n": 1_234_567, "pids": "all", "f32": True,
         "alphas": True, "outside": 0.01},
        # one process's incoming partons only: a flavour subset out of order
        {"name": "xfxq2_subset", "op": "xfxq2", "grid": "three", "n": 3_000_001, "pids": "21,2,-2,1,-1",
         "f32": False, "alphas": False, "outside": 0.01},
        # the running coupling on its own, at every point of a large sample
        {"name": "alphas_1e7", "op": "alphas", "grid": "three", "n": 10_000_000},
        # an error set: many members, uneven requests, one plan replayed
        {"name": "batched_101", "op": "batched", "members": 101, "requests": 200, "log10_n": 4.5, "layout": 2003,
         "f64": False},
        # predictions of 100 members: evaluation on the table's x grid, then the table contraction
        {"name": "members_fk_100", "op": "members", "members": 100, "rows": 1024, "layout": 0},
        # Monte-Carlo integration, chunk by chunk: both lookups, alpha_s and the sum in one call
        {"name": "mc_fused_1e6", "op": "mc", "n": 1_000_000, "f32": False},
        {"name": "mc_fused_f32", "op": "mc", "n": 300_007, "f32": True},
        # the network in place of the grid, at a large sample (drawn weights: the time does not depend on them)
        {"name": "surrogate_1e7", "op": "surrogate", "n": 10_000_000, "pids": "all"},
        # training the network: Adam steps on a resident sample
        {"name": "surrogate_train", "op": "train", "samples": 400_000, "batch": 4096, "steps": 100},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _pid_text(rng, stored):
    if rng.random() < 0.5:
        return "all"
    return ",".join(str(p) for p in rng.sample(stored, rng.randint(1, len(stored))))


def draw(rng):
    op = rng.choice(["xfxq2"] * 5 + ["alphas", "batched", "members", "mc", "mc", "surrogate", "train"])
    if op == "xfxq2":
        grid = rng.choice(["one", "three"])
        return {"op": op, "grid": grid, "n": _log_int(rng, 100, 10_000_000), "pids": _pid_text(rng, PIDS[grid]),
                "f32": rng.random() < 0.5, "alphas": rng.random() < 0.5, "outside": rng.choice([0.0, 0.01, 0.03])}
    if op == "alphas":
        return {"op": op, "grid": rng.choice(["one", "three"]), "n": _log_int(rng, 1000, 10_000_000)}
    if op == "batched":
        return {"op": op, "members": rng.randint(1, 101), "requests": rng.randint(1, 200),
                "log10_n": rng.uniform(3.0, 4.5), "layout": rng.randint(1, 10 ** 6), "f64": rng.random() < 0.3}
    if op == "members":
        return {"op": op, "members": _log_int(rng, 10, 400), "rows": _log_int(rng, 30, 1024), "layout": 0}
    if op == "mc":
        return {"op": op, "n": _log_int(rng, 1000, 2_000_000), "f32": rng.random() < 0.5}
    if op == "surrogate":
        return {"op": op, "n": _log_int(rng, 1000, 10_000_000), "pids": _pid_text(rng, PIDS["one"])}
    return {"op": op, "samples": 200_000, "batch": 16 * _log_int(rng, 16, 512), "steps": rng.randint(20, 100)}


# ---------------------------------------------------------------------------------------
# Inputs


class Grid:
    """Knots and values of one member, and the loaded member while it lives."""

    def __init__(self, kind, rng, base=None):
        self.kind, self.pids = kind, PIDS[kind]
        xk = X_MIN[kind] ** (1.0 - np.arange(N_X[kind]) / (N_X[kind] - 1.0))
        xk[-1] = 1.0
        e = Q_EDGES[kind]
        self.xk, self.qk, self.values = [], [], []
        if base is None:   # x f = x^a (1-x)^b (1 + c sqrt(x) + d x)(1 + e ln(Q^2 / 2.7)) per flavour
            par = rng.uniform([-0.3, 2.0, -1.0, -1.0, -0.1], [0.8, 6.0, 2.0, 2.0, 0.1], (len(self.pids), 5))
        for k in range(len(e) - 1):
            q = np.exp(np.linspace(math.log(e[k]), math.log(e[k + 1]), N_Q[kind]))
            q[0], q[-1] = e[k], e[k + 1]
            q2 = q * q
            if base is None:
                x, l = xk[:, None, None], np.log(q2 / 2.7)[None, :, None]
                v = x ** par[:, 0] * (1 - x) ** par[:, 1] * (1 + par[:, 2] * np.sqrt(x) + par[:, 3] * x) * (1 + par[:, 4] * l)
                if kind == "three":   # heavy flavours vanish below their thresholds
                    for j, p in enumerate(self.pids):
                        if (abs(p) == 4 and k < 1) or (abs(p) == 5 and k < 2) or abs(p) == 6:
                            v[:, :, j] = 0.0
            else:                     # a replica of another member
                v = base.values[k] * np.exp(0.05 * rng.standard_normal(base.values[k].shape))
            self.xk.append(xk)
            self.qk.append(q2)
            self.values.append(np.ascontiguousarray(v))
        self.id = None

    def load(self):
        self.id = pdfmi.load_grid(self.xk, self.qk, self.values, self.pids)
        return self

    def __del__(self):
        if self.id is not None:
            pdfmi.unload(self.id)

    def request(self, text):
        return list(self.pids) if text == "all" else [int(p) for p in text.split(",")]

    def columns(self, pids):
        return [self.pids.index(p) if p in self.pids else -1 for p in pids]


def _alphas_table(kind):
    e = Q_EDGES[kind]
    q2 = np.concatenate([np.exp(np.linspace(math.log(a), math.log(b), N_Q[kind])) ** 2 for a, b in zip(e, e[1:])])
    for k in range(len(e) - 1):       # a threshold's knot is repeated exactly
        q2[k * N_Q[kind]], q2[(k + 1) * N_Q[kind] - 1] = e[k] ** 2, e[k + 1] ** 2
    return q2, 0.118 / (1.0 + 0.02 * np.log(8315.0 / q2))


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _loguniform(gen, n, lo, hi):
    u = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64)
    return (math.log(lo) + u * (math.log(hi) - math.log(lo))).exp_().clamp_(max=math.nextafter(hi, 0.0))


def _points(kind, gen, n, outside):
    """x and Q^2, log-uniform over the grid, a share of them outside it: a
    quarter each below x, below Q, above Q and in the corners."""
    e = Q_EDGES[kind]
    x, q = _loguniform(gen, n, X_MIN[kind], 1.0), _loguniform(gen, n, e[0], e[-1])
    if outside:
        out = torch.rand(n, generator=gen, device=DEV) < outside
        where = torch.randint(0, 5, (n,), generator=gen, device=DEV)
        lowx = out & ((where == 0) | (where >= 3))
        x = torch.where(lowx, _loguniform(gen, n, 0.01 * X_MIN[kind], X_MIN[kind]), x)
        q = torch.where(out & ((where == 1) | (where == 3)), _loguniform(gen, n, 0.5 * e[0], e[0]), q)
        q = torch.where(out & ((where == 2) | (where == 4)), _loguniform(gen, n, e[-1] * (1 + 1e-9), 10 * e[-1]), q)
    return x, q * q


def _layout(case):
    """Requests of a batched case: (member, flavours, points), uneven."""
    r = np.random.default_rng(case["layout"])
    reqs = []
    for _ in range(case["requests"]):
        n = int(round(10.0 ** np.clip(r.normal(case["log10_n"], 0.75), 3.0, 6.0)))
        pids = [int(p) for p in r.permutation(PIDS["one"])[:int(r.integers(1, 12))]]
        reqs.append((int(r.integers(0, case["members"])), pids, n))
    return reqs


def _offsets(sizes):
    """Start of each of a sequence of arrays in one buffer, 64 elements aligned, and the buffer's size."""
    at = np.concatenate([[0], np.cumsum([(s + 63) // 64 * 64 for s in sizes])])
    return [int(a) for a in at[:-1]], int(at[-1])


def _members(case, seed):
    rng = np.random.default_rng(seed)
    base = Grid("one", rng)
    return [base] + [Grid("one", rng, base) for _ in range(case["members"] - 1)]


def _network(seed):
    """Flat parameters of the network, Glorot-uniform with small biases."""
    r = np.random.default_rng([int(seed), 7])
    parts = [r.uniform(-1, 1, s).astype(np.float32) * np.float32(math.sqrt(6.0 / sum(s)) if len(s) == 2 else 0.1)
             for s in SUR_SHAPES]
    return np.concatenate([p.ravel() for p in parts])


class Network:
    def __init__(self, grid, seed):
        self.grid = grid              # kept: the network falls back to its grid
        self.sur = pdfmi.Surrogate(grid.id, seed=int(seed))
        self.sur.set_params(_network(seed))

    def __del__(self):
        self.sur.destroy()


class Plan:
    def __init__(self, requests, f64, keep, tile=None):
        self.keep = keep
        self.plan = pdfmi.BatchPlan(requests, out_f64=f64)
        t, v = (tile, 1) if tile else self.plan.autotune(reps=2)
        self.plan.configure(tile_points=t, vector_cols=v, use_graph=1)

    def __del__(self):
        self.plan.destroy()


def prepare(case, seed):
    op, gen, rng = case["op"], _gen(seed), np.random.default_rng(seed)
    s = {"op": op, "case": dict(case)}
    if op in ("xfxq2", "alphas"):
        pdfmi.load_alphas(*_alphas_table(case["grid"]))
        s["x"], s["q2"] = _points(case["grid"], gen, case["n"], case.get("outside", 0.0))
        s["as"] = torch.empty(case["n"], dtype=torch.float64, device=DEV)
        if op == "xfxq2":
            s["grid"] = Grid(case["grid"], rng).load()
            s["pids"] = s["grid"].request(case["pids"])
            s["out"] = torch.empty((case["n"], len(s["pids"])), device=DEV,
                                   dtype=torch.float32 if case["f32"] else torch.float64)
    elif op == "batched":
        reqs, grids = _layout(case), [g.load() for g in _members(case, seed)]
        at, size = _offsets([n for _, _, n in reqs])
        ot, osize = _offsets([n * len(p) for _, p, n in reqs])
        x, q2 = _points("one", gen, size, 0.0)
        s["out"] = torch.zeros(osize, device=DEV, dtype=torch.float64 if case["f64"] else torch.float32)
        todo = [(grids[m].id, p, x[a:a + n], q2[a:a + n], s["out"][o:o + n * len(p)].view(n, len(p)))
                for (m, p, n), a, o in zip(reqs, at, ot)]
        s["plan"] = Plan(todo, case["f64"], (grids, x, q2))
    elif op == "members":
        grids = [g.load() for g in _members(case, seed)]
        x, q2 = _fk_points()
        s["F"] = torch.empty((case["members"], FK_NX, 13), dtype=torch.float64, device=DEV)
        s["plan"] = Plan([(g.id, PIDS["three"], x, q2, f) for g, f in zip(grids, s["F"])], True, (grids, x, q2), 2048)
        s["table"] = torch.rand((case["rows"], FK_NX * 13), generator=gen, dtype=torch.float64, device=DEV)
        s["T"] = torch.empty((case["members"], case["rows"]), dtype=torch.float64, device=DEV)
    elif op == "mc":
        pdfmi.load_alphas(*_alphas_table("one"))
        s["grid"] = Grid("one", rng).load()
        s["x1"], s["x2"], s["q2"] = _mc_points(case, gen)
        s["ws"] = pdfmi.mc_workspace(case["n"], DEV)
        s["sum"] = torch.empty(1, dtype=torch.float64, device=DEV)
    elif op == "surrogate":
        s["x"], s["q2"] = _points("one", gen, case["n"], 0.0)
        s["net"] = Network(Grid("one", rng).load(), seed)
        s["pids"] = s["net"].grid.request(case["pids"])
        s["out"] = torch.empty((case["n"], len(s["pids"])), dtype=torch.float32, device=DEV)
    else:
        s["net"] = Network(Grid("one", rng).load(), seed)
        s["net"].sur.set_data(*_points("one", gen, case["samples"], 0.0))
        s["loss"] = torch.empty(case["steps"], dtype=torch.float32, device=DEV)
    return s


def _fk_points():
    x = torch.logspace(-6, 0, FK_NX, dtype=torch.float64, device=DEV).clamp_(1e-6, 1.0)
    return x, torch.full((FK_NX,), FK_Q * FK_Q, dtype=torch.float64, device=DEV)


def _mc_points(case, gen):
    x1, x2 = (_loguniform(gen, case["n"], 1e-5, 1.0) for _ in range(2))
    return x1, x2, _loguniform(gen, case["n"], 10.0, 1e3) ** 2


def run(s):
    op, case = s["op"], s["case"]
    if op == "xfxq2":
        if case["alphas"]:
            pdfmi.xfxq2_alphas(s["grid"].id, s["pids"], s["x"], s["q2"], out=s["out"], alphas_out=s["as"],
                               f32=case["f32"])
            return s["out"], s["as"]
        return (pdfmi.xfxq2_f32 if case["f32"] else pdfmi.xfxq2)(s["grid"].id, s["pids"], s["x"], s["q2"], out=s["out"])
    if op == "alphas":
        return pdfmi.alphas_q2(s["q2"], out=s["as"])
    if op == "batched":
        s["plan"].plan.run()
        return s["out"]
    if op == "members":
        s["plan"].plan.run()
        pdfmi.fk_contract(s["F"], s["table"], out=s["T"])
        return s["F"], s["T"]
    if op == "mc":
        return pdfmi.mc_fused(s["grid"].id, PIDS["three"], s["x1"], s["x2"], s["q2"], f32=case["f32"],
                              workspace=s["ws"], out=s["sum"])
    if op == "surrogate":
        return s["net"].sur.xfxq2(s["x"], s["q2"], pids=s["pids"], out=s["out"])
    s["net"].sur.train(case["steps"], case["batch"], 3e-3, 3e-5, 20_000, loss_out=s["loss"])
    return s["loss"], s["net"].sur.params()   # the weights a program reads back after its steps


def work(case):
    """Inputs read once, outputs written once; operations: per PDF value the
    20 multiply-adds of the 4x4 stencil, per point two logarithms and sixteen
    weights (about 100), per alpha_s about 60."""
    op = case["op"]
    grid = {"one": 50 * 30 * 11 * 8, "three": 3 * 196 * 17 * 13 * 8}
    if op == "xfxq2":
        P = len(PIDS[case["grid"]]) if case["pids"] == "all" else len(case["pids"].split(","))
        n, w = case["n"], 4 if case["f32"] else 8
        return {"bytes": n * (16 + w * P + 8 * case["alphas"]) + grid[case["grid"]] * w // 8,
                "flops": n * (40 * P + 100 + 60 * case["alphas"])}
    if op == "alphas":
        return {"bytes": 16 * case["n"], "flops": 60 * case["n"]}
    if op == "batched":
        w, reqs = 8 if case["f64"] else 4, _layout(case)
        used = len({m for m, _, _ in reqs})
        return {"bytes": sum(n * (16 + w * len(p)) for _, p, n in reqs) + used * grid["one"] * w // 8,
                "flops": sum(n * (40 * len(p) + 100) for _, p, n in reqs)}
    if op == "members":
        m, K = case["members"], FK_NX * 13
        return {"bytes": m * grid["one"] + 16 * FK_NX + 8 * (2 * m * K + case["rows"] * K + m * case["rows"]),
                "flops": m * FK_NX * (40 * 11 + 100) + 2 * m * K * case["rows"]}
    if op == "mc":
        return {"bytes": 24 * case["n"] + grid["one"] // (2 if case["f32"] else 1),
                "flops": case["n"] * (2 * 11 * 40 + 2 * 13 + 210)}
    mac = 2 * 64 + 2 * 64 * 64 + 64 * 16
    if op == "surrogate":
        P = len(PIDS["one"]) if case["pids"] == "all" else len(case["pids"].split(","))
        return {"bytes": case["n"] * (16 + 4 * P), "flops": case["n"] * (2 * mac + 3 * 64 * 4)}
    rows, par = case["steps"] * case["batch"], sum(int(np.prod(s)) for s in SUR_SHAPES)
    return {"bytes": 72 * rows + case["steps"] * 4 * (6 * par), "flops": 6 * mac * rows}


# ---------------------------------------------------------------------------------------
# The same results in plain torch, FP64


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def _stencil(knots, v):
    """Cell i of each v, its parameter u in ln v, and the weights of knots
    i-1..i+2 (indices clamped; their weight is 0 beyond the table): cubic
    Hermite, slopes the mean of the adjacent secants, one-sided at the ends."""
    n = len(knots)
    i = (torch.searchsorted(knots, v, right=True) - 1).clamp_(0, n - 2)
    D = (knots[1:] / knots[:-1]).log()
    Di = D[i]
    u = (v / knots[i]).log() / Di
    L, R = i > 0, i < n - 2
    hl = torch.where(L, 0.5 * Di / D[(i - 1).clamp(min=0)], 0.0)
    hr = torch.where(R, 0.5 * Di / D[(i + 1).clamp(max=n - 2)], 0.0)
    w = 1.0 - u
    h00, h10, h01, h11 = w * w * (1 + 2 * u), u * w * w, u * u * (3 - 2 * u), -w * u * u
    a1, b0 = torch.where(L, 0.5, 1.0), torch.where(R, -0.5, -1.0)
    W = torch.stack([-hl * h10, h00 + h10 * (hl - a1) + h11 * b0, h01 + h10 * a1 + h11 * (-b0 - hr), hr * h11], 1)
    idx = torch.stack([(i + d).clamp(0, n - 1) for d in (-1, 0, 1, 2)], 1)
    return idx, W, u


def _below(f0, f1, s):
    ok = (f0 > 1e-3) & (f1 > 1e-3)
    return torch.where(ok, f0 * (torch.where(ok, f1 / f0, 1.0)) ** s, f0 + s * (f1 - f0))


def _above(f0, f1, s):
    ok = (f0 > 1e-3) & (f1 > 1e-3)
    return torch.where(ok, f1 * (torch.where(ok, f1 / f0, 1.0)) ** s, f1 + s * (f1 - f0))


def _xf_block(grid, x, q2):
    """x f of every stored flavour at points of any region."""
    out = torch.empty((len(x), len(grid.pids)), dtype=torch.float64, device=DEV)
    last = len(grid.qk) - 1
    for k in range(last + 1):
        xk, qk, V = _t(grid.xk[k]), _t(grid.qk[k]), _t(grid.values[k])
        sel = ((q2 >= qk[0]) | (k == 0)) & ((q2 < qk[-1]) | (k == last))
        at = sel.nonzero()[:, 0]
        xs, qs = x[at], q2[at]
        xi, xw, ux = _stencil(xk, xs)
        qi, qw, uq = _stencil(qk, qs)
        lowx, lowq, highq = xs < xk[0], qs < qk[0], qs > qk[-1]
        rows = torch.einsum("nb,nabc->nac", qw, V[xi[:, :, None], qi[:, None, :]])
        v = (xw[:, :, None] * rows).sum(1)
        if bool((lowx | lowq | highq).any()):
            p = (lowx & ~lowq & ~highq).nonzero()[:, 0]
            v[p] = _below(rows[p, 1], rows[p, 2], ux[p, None])   # its cell is the first: rows x_0, x_1
            p = (lowq | highq).nonzero()[:, 0]
            r0 = torch.where(lowq[p], 0, len(qk) - 2)
            f = []
            for r in (r0, r0 + 1):                               # x first, on both anchor rows
                inside = (xw[p, :, None] * V[xi[p], r[:, None]]).sum(1)
                f.append(torch.where(lowx[p, None], _below(V[0, r], V[1, r], ux[p, None]), inside))
            f0, f1 = f
            r = (qs[p] / qk[0])[:, None]
            ok = (f0 > 1e-5) & (f1 > 1e-5) & (xs[p, None] <= 0.9)
            gamma = torch.where(ok, f1 / torch.where(ok, f0, 1.0), 1.0).log() / (qk[1] / qk[0]).log()
            low = f0 * torch.where(ok, r ** (gamma * r + 1.0 - r), r)
            v[p] = torch.where(lowq[p, None], low, _above(f0, f1, uq[p, None] - 1.0))
        out[at] = v
    return out


def _xf(grid, pids, x, q2):
    cols = grid.columns(pids)
    out = torch.zeros((len(x), len(pids)), dtype=torch.float64, device=DEV)
    have = [j for j, c in enumerate(cols) if c >= 0]
    take = torch.tensor([cols[j] for j in have], device=DEV)
    for a in range(0, len(x), 500_000):
        out[a:a + 500_000, have] = _xf_block(grid, x[a:a + 500_000], q2[a:a + 500_000])[:, take]
    return out


def _alphas(kind, q2):
    k, v = (_t(a) for a in _alphas_table(kind))
    n, out = N_Q[kind], torch.empty_like(q2)
    for s in range(len(k) // n):
        ks, vs = k[s * n:(s + 1) * n], v[s * n:(s + 1) * n]
        at = (((q2 >= ks[0]) | (s == 0)) & ((q2 < ks[-1]) | (s == len(k) // n - 1))).nonzero()[:, 0]
        i, w, _ = _stencil(ks, q2[at].clamp(float(ks[0]), float(ks[-1])))
        out[at] = (w * vs[i]).sum(1)
    return out


def _envelope(grid):
    """ln of the x knots and, per knot, the signed value of largest magnitude over Q^2 with its slope in ln x."""
    V = _t(grid.values[0])
    e = V.gather(1, V.abs().argmax(1, keepdim=True))[:, 0]
    lx = _t(grid.xk[0]).log()
    sec = (e[1:] - e[:-1]) / (lx[1:] - lx[:-1])[:, None]
    return lx, e, torch.cat([sec[:1], 0.5 * (sec[1:] + sec[:-1]), sec[-1:]])


def _at_envelope(env, x):
    lx, e, d = env
    l = x.log()
    i = (torch.searchsorted(lx, l, right=True) - 1).clamp_(0, len(lx) - 2)
    D = lx[i + 1] - lx[i]
    t = ((l - lx[i]) / D).clamp(0, 1)
    h = [(1 - t) ** 2 * (1 + 2 * t), t * (1 - t) ** 2 * D, t * t * (3 - 2 * t), -(1 - t) * t * t * D]
    return h[0][:, None] * e[i] + h[1][:, None] * d[i] + h[2][:, None] * e[i + 1] + h[3][:, None] * d[i + 1]


def _in_domain(grid, x, q2):
    xk, qk = grid.xk[0], grid.qk[0]
    return (x >= xk[1]) & (x < xk[-2]) & (q2 >= qk[1]) & (q2 < qk[-2])


def _net_inputs(grid, x, q2):
    xk, qk = grid.xk[0], grid.qk[0]
    u = 2.0 * (x.log() - math.log(xk[0])) / (math.log(xk[-1]) - math.log(xk[0])) - 1.0
    return torch.stack([u, 2.0 * (q2.log() - math.log(qk[0])) / (math.log(qk[-1]) - math.log(qk[0])) - 1.0], 1)


def _split(flat):
    out, o = [], 0
    for s in SUR_SHAPES:
        n = int(np.prod(s))
        out.append(flat[o:o + n].reshape(s))
        o += n
    return out


def _forward(p, h):
    for layer in range(3):
        h = torch.tanh(h @ p[2 * layer].T + p[2 * layer + 1])
    return h @ p[6].T + p[7]


def _train_exact(case, grid, seed):
    x, q2 = _points("one", _gen(seed), case["samples"], 0.0)
    keep = _in_domain(grid, x, q2)
    x, q2 = x[keep], q2[keep]
    T = torch.zeros((len(x), 16), dtype=torch.float64, device=DEV)
    e = _at_envelope(_envelope(grid), x)
    T[:, :11] = torch.where(e != 0, _xf(grid, grid.pids, x, q2) / e, 0.0)
    h = _net_inputs(grid, x, q2)
    p = _t(_network(seed).astype(np.float64)).requires_grad_(True)
    m, v, B, losses = torch.zeros_like(p), torch.zeros_like(p), case["batch"], []
    for step in range(case["steps"]):
        b = (step % (len(x) // B)) * B
        loss = ((_forward(_split(p), h[b:b + B]) - T[b:b + B]) ** 2).mean()
        g, = torch.autograd.grad(loss, p)
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        lr = 3e-5 + 0.5 * (3e-3 - 3e-5) * (1 + math.cos(math.pi * min(1.0, step / 20_000)))
        with torch.no_grad():
            p -= lr * (m / (1 - 0.9 ** (step + 1))) / ((v / (1 - 0.999 ** (step + 1))).sqrt() + 1e-8)
        losses.append(float(loss))
    return _t(losses), p.detach().cpu().numpy()


def exact(case, seed):
    op, gen, rng = case["op"], _gen(seed), np.random.default_rng(seed)
    if op in ("xfxq2", "alphas"):
        x, q2 = _points(case["grid"], gen, case["n"], case.get("outside", 0.0))
        if op == "alphas":
            return _alphas(case["grid"], q2)
        grid = Grid(case["grid"], rng)
        out = _xf(grid, grid.request(case["pids"]), x, q2)
        return (out, _alphas(case["grid"], q2)) if case["alphas"] else out
    if op == "batched":
        reqs, grids = _layout(case), _members(case, seed)
        at, size = _offsets([n for _, _, n in reqs])
        ot, osize = _offsets([n * len(p) for _, p, n in reqs])
        x, q2 = _points("one", gen, size, 0.0)
        out = torch.zeros(osize, dtype=torch.float64, device=DEV)
        for (m, p, n), a, o in zip(reqs, at, ot):
            out[o:o + n * len(p)] = _xf(grids[m], p, x[a:a + n], q2[a:a + n]).reshape(-1)
        return out
    if op == "members":
        x, q2 = _fk_points()
        F = torch.stack([_xf(g, PIDS["three"], x, q2) for g in _members(case, seed)])
        table = torch.rand((case["rows"], FK_NX * 13), generator=gen, dtype=torch.float64, device=DEV)
        return F, F.reshape(case["members"], -1) @ table.T
    if op == "mc":
        grid = Grid("one", rng)
        x1, x2, q2 = _mc_points(case, gen)
        lum = (_xf(grid, grid.pids, x1, q2) * _xf(grid, grid.pids, x2, q2)).sum(1)
        return (_alphas("one", q2) * lum).sum().reshape(1)
    grid = Grid("one", rng)
    if op == "train":
        return _train_exact(case, grid, seed)
    x, q2 = _points("one", gen, case["n"], 0.0)
    pids = grid.request(case["pids"])
    cols = torch.tensor(grid.columns(pids), device=DEV)
    p, env = _split(_t(_network(seed).astype(np.float64))), _envelope(grid)
    out = torch.empty((case["n"], len(pids)), dtype=torch.float64, device=DEV)
    for a in range(0, case["n"], 500_000):
        xs, qs = x[a:a + 500_000], q2[a:a + 500_000]
        y = _forward(p, _net_inputs(grid, xs, qs))[:, :11] * _at_envelope(env, xs)
        y = torch.where(_in_domain(grid, xs, qs)[:, None], y, _xf_block(grid, xs, qs))
        out[a:a + 500_000] = y[:, cols]
    return out
