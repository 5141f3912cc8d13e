"""The work a user of this library has it do, as cases that can be timed.

Every case goes through the public entry points of the ctypes binding: whole
solves, a solver advanced step by step, a server's request mix, and the
step-level calls that stand on their own (the matrix exponential, its action,
the column compression, the Riccati update).  ``listed()`` names the cases,
``draw()`` gives further ones of the same ranges, ``prepare()`` makes a case's
inputs and the handle a program keeps, ``run()`` is one pass, ``work()`` the
bytes and operations that pass cannot do without, and ``exact()`` the same
results from plain dense 64-bit arithmetic.

Results of a solve are compared as P = L D L^T (or as the feedback gain
R^-1 B^T P that an LQR program reads), because L itself is only determined up
to the signs of its columns and rotations among near-equal eigenvalues.
"""
import math
import time

import numpy as np
import torch

from paper_1805_08990_amd import _binding as b


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _solve(name, **kw):
    c = {"name": name, "what": "solve", "kind": "dre", "op": "laplace", "nx": 32, "m": 2, "p": 3, "steps": 20,
         "h": 1e-3, "scheme": "strang", "split": "F12", "precision": "fp64", "action": "dense", "S": False,
         "tol": 1e-10}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest solve: 16 x 16 Laplacian, plain Strang splitting, one
        # output row; launches and host round trips are all of it
        _solve("solve_dle_256", kind="dle", nx=16, m=0, p=1, steps=100, split="F1F2", tol=1e-12),
        # an ordinary solve of a served size, operator setup included
        _solve("solve_dre_1024", nx=32, m=2, p=4, steps=50),
        # generalized Riccati equation (S P S^T) on a ragged grid: wide
        # compressions of [L, S L, S^2 L]
        _solve("solve_gdre_2025", nx=45, m=1, p=1, steps=10, S=True),
        # a nonsymmetric operator in the mixed-precision mode: eight dense
        # exponentials and split-BF16 products
        _solve("solve_nonsym_mixed_1030", op="nonsym", nx=1030, m=3, p=2, steps=10, h=1e-2, precision="mixed"),
        # stepping a controller whose operator is set up once, reading its
        # gain: dense FP64 products at 96 x 96
        {"name": "steps_fp64_9216", "what": "steps", "nx": 96, "m": 4, "p": 8, "warm": 20, "steps": 5, "h": 1e-3,
         "precision": "fp64", "action": "dense"},
        # the headline size, split-BF16 products
        {"name": "steps_mixed_16384", "what": "steps", "nx": 128, "m": 4, "p": 8, "warm": 20, "steps": 5, "h": 1e-3,
         "precision": "mixed", "action": "dense"},
        # the headline size, Leja action on the sparse operator
        {"name": "steps_leja_16384", "what": "steps", "nx": 128, "m": 4, "p": 8, "warm": 20, "steps": 5, "h": 1e-3,
         "precision": "fp64", "action": "leja"},
        # the dense exponential alone (the setup of every dense solver, and a
        # call of its own): diffusion-reaction at 64 x 64
        {"name": "expm_4096", "what": "expm", "op": "reaction", "n": 4096, "t": 5e-4},
        # the exponential's action on a block, CSR operator: expleja as a call
        # of its own
        {"name": "expmv_16384x8", "what": "expmv", "nx": 128, "cols": 8, "t": 5e-4},
        # compressing the difference of two solutions (indefinite D)
        {"name": "compress_4096x96", "what": "compress", "n": 4096, "k": 96, "indefinite": True, "tol": 1e-10},
        # one closed-form Riccati update on a small factor: the smallest call
        {"name": "riccati_1024", "what": "riccati", "n": 1024, "r": 40, "m": 2, "t": 1e-3},
        # a burst of requests to a warm server
        {"name": "serve_burst_12", "what": "serve", "nx": 32, "nx2": 48, "count": 12, "steps": 25, "slots": 8,
         "precision": "mixed"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["solve", "solve", "solve", "steps", "steps", "expm", "expmv", "compress", "riccati", "serve"])
    if what == "solve":
        form = rng.choice(["dle", "dle", "dre", "dre", "gdre", "nonsym", "mass", "leja"])
        c = _solve("", nx=rng.randint(9, 45), m=rng.randint(1, 4), p=rng.randint(1, 8), steps=rng.randint(5, 30),
                   scheme=rng.choice(["strang", "strang", "lie"]), split=rng.choice(["F12", "F12", "F1F2"]),
                   precision=rng.choice(["fp64", "mixed"]), h=rng.choice([1e-3, 2e-3, 5e-3]))
        if form == "dle":
            c.update(kind="dle", m=0)
        elif form == "gdre":
            c.update(S=True, split="F12", m=1, p=rng.randint(1, 2), steps=rng.randint(3, 10), precision="fp64")
        elif form == "nonsym":
            c.update(op="nonsym", nx=_log_int(rng, 90, 1100), h=1e-2, steps=rng.randint(5, 15))
        elif form == "mass":
            c.update(op="mass", nx=rng.randint(8, 24), precision="fp64")
        elif form == "leja":
            c.update(action="leja", precision="fp64")
        del c["name"]
        return c
    if what == "steps":
        action = rng.choice(["dense", "leja"])
        return {"what": "steps", "nx": rng.randint(24, 128 if action == "leja" else 80), "m": rng.randint(1, 6),
                "p": rng.randint(1, 8), "warm": rng.randint(5, 20), "steps": rng.randint(1, 6),
                "h": rng.choice([5e-4, 1e-3, 2e-3]), "action": action,
                "precision": "fp64" if action == "leja" else rng.choice(["fp64", "mixed"])}
    if what == "expm":
        return {"what": "expm", "op": rng.choice(["reaction", "convection"]), "n": _log_int(rng, 60, 4096),
                "t": rng.choice([1e-5, 1e-4, 5e-4, 1e-3])}
    if what == "expmv":
        return {"what": "expmv", "nx": rng.randint(16, 128), "cols": _log_int(rng, 1, 128),
                "t": rng.choice([1e-4, 5e-4, 1e-3])}
    if what == "compress":
        return {"what": "compress", "n": _log_int(rng, 300, 4096), "k": _log_int(rng, 8, 200),
                "indefinite": rng.choice([True, False]), "tol": rng.choice([1e-8, 1e-10, 1e-12])}
    if what == "riccati":
        return {"what": "riccati", "n": _log_int(rng, 200, 16384), "r": _log_int(rng, 4, 200),
                "m": rng.randint(1, 8), "t": 1e-3}
    return {"what": "serve", "nx": rng.randint(16, 40), "nx2": rng.randint(24, 48), "count": rng.randint(4, 12),
            "steps": rng.randint(10, 25), "slots": rng.choice([2, 4, 8]), "precision": rng.choice(["fp64", "mixed"])}


# --------------------------------------------------------------------------
# problem data
# --------------------------------------------------------------------------
def _tridiag(nx):
    dx = 1.0 / (nx + 1)
    t = np.diag(np.full(nx, -2.0)) + np.diag(np.ones(nx - 1), 1) + np.diag(np.ones(nx - 1), -1)
    return t / (dx * dx)


def _laplace_csr(nx):
    """Five-point Dirichlet Laplacian on the nx x nx interior grid, x fastest."""
    n, s = nx * nx, float((nx + 1) ** 2)
    k = np.arange(n)
    i, j = k % nx, k // nx
    cols = np.stack([k - nx, k - 1, k, k + 1, k + nx], axis=1)
    vals = np.tile(np.array([s, s, -4.0 * s, s, s]), (n, 1))
    keep = np.stack([j > 0, i > 0, np.ones(n, bool), i < nx - 1, j < nx - 1], axis=1)
    rowptr = np.concatenate([[0], np.cumsum(keep.sum(axis=1))]).astype(np.int64)
    return rowptr, cols[keep].astype(np.int64), np.ascontiguousarray(vals[keep])


def _laplace(nx):
    rowptr, cols, vals = _laplace_csr(nx)
    A = np.zeros((nx * nx, nx * nx), order="F")
    A[np.repeat(np.arange(nx * nx), np.diff(rowptr)), cols] = vals
    return A


def _mass_pair(nx):
    """Bilinear elements on a tensor mesh graded towards two sides: (A, M)."""
    x = (np.arange(nx + 2) / (nx + 1.0)) ** 1.3
    he = np.diff(x)
    off = np.arange(nx - 1)
    M1 = np.diag((he[:-1] + he[1:]) / 3.0)
    K1 = np.diag(1.0 / he[:-1] + 1.0 / he[1:])
    M1[off, off + 1] = M1[off + 1, off] = he[1:-1] / 6.0
    K1[off, off + 1] = K1[off + 1, off] = -1.0 / he[1:-1]
    return np.asfortranarray(-(np.kron(K1, M1) + np.kron(M1, K1))), np.asfortranarray(np.kron(M1, M1))


def _quadrants(nx, m, rng):
    """Indicators of the four quadrants; further inputs act on random patches."""
    g = (np.arange(nx) + 1.0) / (nx + 1)
    x, y = np.tile(g, nx), np.repeat(g, nx)
    cols = [(x < 0.5) & (y < 0.5), (x >= 0.5) & (y < 0.5), (x < 0.5) & (y >= 0.5), (x >= 0.5) & (y >= 0.5)][:m]
    while len(cols) < m:
        cols.append((abs(x - rng.uniform(0.2, 0.8)) < 0.2) & (abs(y - rng.uniform(0.2, 0.8)) < 0.2))
    return np.asfortranarray(np.stack(cols, axis=1).astype(np.float64))


def _problem(c, seed, dense=True):
    """Host arrays of one solve: A (dense, or None), M, B, C, R, S."""
    rng = np.random.default_rng(seed)
    op = c.get("op", "laplace")
    n = c["nx"] if op == "nonsym" else c["nx"] ** 2
    d = {"n": n, "A": None, "M": None, "B": None, "R": None, "S": None}
    if op == "nonsym":
        d["A"] = np.asfortranarray(rng.standard_normal((n, n)) / math.sqrt(n) - 1.5 * np.eye(n))
    elif op == "mass":
        d["A"], d["M"] = _mass_pair(c["nx"])
    elif dense:
        d["A"] = _laplace(c["nx"])
    d["C"] = np.asfortranarray(rng.standard_normal((c["p"], n)) / math.sqrt(n))
    if c.get("kind", "dre") == "dre":
        d["B"] = (np.asfortranarray(rng.standard_normal((n, c["m"]))) if op == "nonsym"
                  else _quadrants(c["nx"], c["m"], rng))
        d["R"] = np.asfortranarray(np.eye(c["m"]) * rng.uniform(0.5, 2.0))
    if c.get("S"):
        S = np.zeros((n, n), order="F")
        k = np.arange(n - 1)
        S[k, k + 1] = S[k + 1, k] = 0.1
        d["S"] = S
    return d


def _options(c, T=None):
    return b.SolveOptions(T=c["steps"] * c["h"] if T is None else T, h=c["h"], tol=c.get("tol", 1e-10),
                          scheme=c.get("scheme", "strang"), split=c.get("split", "F12"), precision=c["precision"],
                          action=c.get("action", "dense"))


def _expm_operator(c, seed):
    """The discretised operator of an expm call on n points: diffusion on a
    near-square grid with a random reaction rate (symmetric), or with a random
    wind (nonsymmetric)."""
    n = c["n"]
    nx = max(2, int(math.isqrt(n)))
    gen = torch.Generator("cuda").manual_seed(seed)
    s = float((nx + 1) ** 2)
    A = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    rate = torch.rand(n, generator=gen, dtype=torch.float64, device="cuda")
    A.diagonal().copy_(-4.0 * s - 100.0 * rate)
    k = torch.arange(n, device="cuda")
    inrow = ((k + 1) % nx != 0).double()[: n - 1]
    A.diagonal(1).copy_(s * inrow)
    A.diagonal(-1).copy_(s * inrow)
    A.diagonal(nx).fill_(s)
    A.diagonal(-nx).fill_(s)
    if c["op"] == "convection":
        wind = 40.0 * (nx + 1) * (torch.rand(n - 1, generator=gen, dtype=torch.float64, device="cuda") - 0.5) * inrow
        A.diagonal(1).add_(wind)
        A.diagonal(-1).sub_(wind)
    return A


def _requests(c, seed):
    """The requests of a burst: (grid side, kind, problem data)."""
    out = []
    for q in range(c["count"]):
        nx = c["nx2"] if q % 3 == 1 else c["nx"]
        kind = "dle" if q % 2 else "dre"
        r = {"nx": nx, "kind": kind, "m": 1 + q % 4, "p": 1 + (3 * q) % 8, "h": 1e-3, "steps": c["steps"] + 2 * (q % 4),
             "precision": c["precision"]}
        out.append((r, _problem(r, 1000 * seed + q, dense=False)))
    return out


def _factors(c, seed):
    """Inputs of a compression: W = [two factors with geometrically graded
    weights], Dhat; of a Riccati update: L, B, R, D."""
    gen = torch.Generator("cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, dtype=torch.float64, device="cuda")

    n = c["n"]
    if c["what"] == "compress":
        k = c["k"]
        W = (normal(k, n) / math.sqrt(n)).t()
        d = 10.0 ** (-13.0 * torch.arange(k, dtype=torch.float64, device="cuda") / k)
        d = d[torch.randperm(k, generator=torch.Generator().manual_seed(seed)).cuda()]
        if c["indefinite"]:
            d = d * torch.where(torch.arange(k, device="cuda") < (k + 1) // 2, 1.0, -1.0)
        return {"W": W, "D": torch.diag(d)}
    r, m = c["r"], c["m"]
    L = (normal(r, n) / math.sqrt(n)).t()
    B = normal(m, n).t()
    d = 10.0 ** (-10.0 * torch.arange(r, dtype=torch.float64, device="cuda") / r)
    R = normal(m, m) * 0.1
    return {"L": L, "B": B, "R": R @ R.t() + torch.eye(m, dtype=torch.float64, device="cuda"), "D": torch.diag(d)}


# --------------------------------------------------------------------------
# one pass through the library
# --------------------------------------------------------------------------
def prepare(case, seed):
    c, what = case, case["what"]
    if what in ("compress", "riccati"):
        return {"case": c, "ctx": b.Context(0), **_factors(c, seed)}
    if what == "expm":
        return {"case": c, "ctx": b.Context(0), "X": _expm_operator(c, seed).t()}
    if what == "expmv":
        gen = torch.Generator("cuda").manual_seed(seed)
        X = torch.randn(c["cols"], c["nx"] ** 2, generator=gen, dtype=torch.float64, device="cuda").t()
        return {"case": c, "ctx": b.Context(0), "A": _laplace_csr(c["nx"]), "X": X}
    ctx = b.Context(0)
    if what == "solve":
        d = _problem(c, seed, dense=c["action"] != "leja")
        if c["action"] == "leja":
            d["A"] = _laplace_csr(c["nx"])
        return {"case": c, "ctx": ctx, **d}
    if what == "steps":
        d = _problem(c, seed, dense=c["action"] != "leja")
        A = _laplace_csr(c["nx"]) if c["action"] == "leja" else d["A"]
        # the horizon is long: a controller that keeps running
        sv = b.Solver(ctx, "dre", _options(c, T=100000 * c["h"]), A, d["C"], B=d["B"], R=d["R"])
        sv.step(c["warm"])
        return {"case": c, "sv": sv}
    srv = ctx.server(32 << 30, max_slots=c["slots"])
    reqs, ids = _requests(c, seed), {}
    for r, _ in reqs:
        if r["nx"] not in ids:
            ids[r["nx"]] = srv.register_operator(_laplace(r["nx"]))
            srv.warm(ids[r["nx"]], 0.5 * r["h"], c["precision"])  # Strang's half step
            srv.warm(ids[r["nx"]], r["h"], c["precision"])        # the whole step of a DLE
    return {"case": c, "ctx": b.Context(0), "srv": srv, "reqs": reqs, "ids": ids}


def _device(x):
    """A column-major host array on the device, as a logical matrix."""
    return torch.from_numpy(x.T).cuda().t()


def _dense_P(ctx, L, D):
    Ld = _device(L)
    return ctx.gemm(ctx.gemm(Ld, _device(D)), Ld, transb="T")


def run(state):
    c, what = state["case"], state["case"]["what"]
    if what == "solve":
        L, D, _ = state["ctx"].solve(c["kind"], _options(c), state["A"], state["C"], B=state["B"], R=state["R"],
                                     S=state["S"], M=state["M"])
        return _dense_P(state["ctx"], L, D)
    if what == "steps":
        state["sv"].step(c["steps"])
        return state["sv"].gain()
    if what == "expm":
        return state["ctx"].expm(state["X"], c["t"])[0]
    if what == "expmv":
        return state["ctx"].expmv_leja(state["A"], c["t"], state["X"])[0]
    if what == "compress":
        ctx = state["ctx"]
        # (the call destroys its factor: a program that keeps W passes a copy)
        L, D = ctx.compress(state["W"].t().clone().t(), state["D"], c["tol"])
        return ctx.gemm(ctx.gemm(L, D), L, transb="T")
    if what == "riccati":
        return state["ctx"].riccati(state["L"], state["B"], state["R"], c["t"], state["D"].clone())
    srv, tickets = state["srv"], []
    for r, d in state["reqs"]:
        tickets.append(srv.submit(state["ids"][r["nx"]], r["kind"], _options(r), d["C"], d["n"], B=d["B"], R=d["R"]))
    got = [None] * len(tickets)
    while any(g is None for g in got):
        for q, tk in enumerate(tickets):
            if got[q] is None:
                got[q] = srv.poll(tk)
        time.sleep(0.0005)
    return [_dense_P(state["ctx"], L, D) for L, D, _, _ in got]


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _rank(p):
    """About the rank P keeps at tolerance 1e-10 with p output rows."""
    return 14 * p + 10


def _expm_products(tnorm):
    """n x n products of scaling and squaring with the [13/13] approximant
    (Higham 2005): powers and polynomials, the solve as 4/3, squarings."""
    return 6 + 4.0 / 3.0 + max(0.0, math.ceil(math.log2(max(tnorm, 1e-9) / 5.37)))


def _step_work(n, r, k, op_bytes, op_flops, half_steps):
    """Half steps: the operator read once and applied to r columns, then the
    compression of k columns to r (Gram matrix and basis change)."""
    return {"bytes": half_steps * (op_bytes + 8.0 * n * (2 * r + k)),
            "flops": half_steps * (op_flops * r + 2.0 * n * k * (k + r))}


def work(case):
    c, what = case, case["what"]
    if what == "riccati":
        return {"bytes": 8.0 * (c["n"] * (c["r"] + c["m"]) + 2 * c["r"] ** 2), "flops": 2.0 * c["n"] * c["r"] * c["m"]}
    if what == "compress":
        n, k = c["n"], c["k"]
        r = k * min(1.0, -math.log10(c["tol"]) / 13.0)
        return {"bytes": 8.0 * n * (k + n), "flops": 2.0 * n * k * (k + r) + 2.0 * n * n * r}
    if what == "expm":
        n = c["n"]
        return {"bytes": 16.0 * n * n, "flops": 2.0 * n ** 3 * _expm_products(c["t"] * 8.0 * n)}
    if what == "expmv":
        n = c["nx"] ** 2
        terms = 10 + 2.5 * c["t"] * 2.0 * n  # degree over all substeps
        return {"bytes": 16.0 * n * c["cols"] + 12.0 * 5 * n, "flops": terms * 12.0 * n * c["cols"]}
    if what == "steps":
        n, r = c["nx"] ** 2, _rank(c["p"])
        eb = {"fp64": 8.0, "mixed": 4.0}[c["precision"]] * n * n if c["action"] == "dense" else 60.0 * n
        ef = 2.0 * n * n if c["action"] == "dense" else 12.0 * n * (10 + 2.5 * c["h"] * n)
        return _step_work(n, r, r + 7 * c["p"], eb, ef, 2 * c["steps"])
    if what == "serve":
        total = {"bytes": 0.0, "flops": 0.0}
        for q in range(c["count"]):
            n = (c["nx2"] if q % 3 == 1 else c["nx"]) ** 2
            r, eb = _rank(1 + (3 * q) % 8), 4.0 if c["precision"] == "mixed" else 8.0
            w = _step_work(n, r, 2 * r, eb * n * n / c["slots"], 2.0 * n * n, 1.5 * (c["steps"] + 2 * (q % 4)))
            total = {k: total[k] + w[k] + 8.0 * n * n for k in total}
        return total
    n = c["nx"] if c["op"] == "nonsym" else c["nx"] ** 2
    r = min(n, _rank(c["p"]))
    tnorm = c["h"] * (4.0 if c["op"] == "nonsym" else 8.0 * n)
    if c["action"] == "leja":
        setup, eb, ef = 0.0, 60.0 * n, 12.0 * n * (10 + 2.5 * c["h"] * n)
    else:
        setup, eb, ef = _expm_products(tnorm) * (8 if c["op"] == "nonsym" else 1), 8.0 * n * n, 2.0 * n * n
    halves = (2 if c["scheme"] == "strang" else 1) * c["steps"]
    w = _step_work(n, r, r + (c["p"] if c["split"] == "F1F2" else 7 * c["p"]), eb, ef, halves)
    if c["S"]:
        w = {k: 3.0 * w[k] for k in w}  # S L, S^2 L and the wider compression
    return {"bytes": w["bytes"] + 16.0 * n * n, "flops": w["flops"] + setup * 2.0 * n ** 3 + 2.0 * n * n * r}


# --------------------------------------------------------------------------
# the same in plain dense 64-bit arithmetic
# --------------------------------------------------------------------------
def _t(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


class _Grid:
    """e^{tA} for the Laplacian through its 1-D factor: exact up to roundoff."""

    def __init__(self, nx):
        self.nx = nx
        w, V = np.linalg.eigh(_tridiag(nx))
        self.w, self.V = _t(w), _t(V)

    def apply(self, t, X):
        e, nx = (self.V * torch.exp(t * self.w)) @ self.V.t(), self.nx
        Y = (e @ X.reshape(nx, -1)).reshape(nx, nx, -1)  # the slow grid direction, then the fast one
        return torch.matmul(e, Y).reshape(X.shape)


class _Dense:
    def __init__(self, AT):
        self.AT, self.known = AT, {}

    def apply(self, t, X):
        if t not in self.known:
            self.known[t] = torch.linalg.matrix_exp(t * self.AT)
        return self.known[t] @ X


def _exact_P(c, d, steps):
    """The scheme on the dense P, without truncation."""
    CT = _t(d["C"].T)
    if c.get("op", "laplace") == "laplace":
        E = _Grid(c["nx"])
    elif d["M"] is not None:
        MT = _t(d["M"].T)
        E = _Dense(torch.linalg.solve(MT, _t(d["A"].T)))
        CT = torch.linalg.solve(MT, CT)
    else:
        E = _Dense(_t(d["A"].T))
    n, h = d["n"], c["h"]
    P = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    quad = {}

    def T1(t, P):
        return E.apply(t, E.apply(t, P).t().contiguous()).t()

    def T12(t, P):
        if t not in quad:
            x, w = np.polynomial.legendre.leggauss(7)
            quad[t] = torch.cat([math.sqrt(0.5 * t * wk) * E.apply(0.5 * t * (xk + 1.0), CT) for xk, wk in zip(x, w)], 1)
        return torch.addmm(T1(t, P), quad[t], quad[t].t())

    def T2(t, P):
        return P + t * (CT @ CT.t())

    B, R = (_t(d["B"]), _t(d["R"])) if d["B"] is not None else (None, None)

    def T3(t, P):
        PB = P @ B
        return P - t * PB @ torch.linalg.solve(R + t * (B.t() @ PB), PB.t())

    def T4(t, P):
        S = _t(d["S"])
        F = S @ P @ S.t()
        return P + t * F + 0.5 * t * t * (S @ F @ S.t())

    inner = ([T3] if c.get("kind", "dre") == "dre" else []) + ([T4] if c.get("S") else [])
    outer = [T12] if c.get("split", "F12") == "F12" else [T1, T2]
    if c.get("scheme", "strang") == "lie":
        seq = [(f, h) for f in outer + inner]
    else:
        flows = outer + inner
        seq = [(f, 0.5 * h) for f in flows[:-1]] + [(flows[-1], h)] + [(f, 0.5 * h) for f in flows[-2::-1]]
    for _ in range(steps):
        for f, t in seq:
            P = f(t, P)
    return P


def exact(case, seed):
    c, what = case, case["what"]
    if what == "solve":
        return _exact_P(c, _problem(c, seed, dense=c["op"] != "laplace"), c["steps"])
    if what == "steps":
        d = _problem(c, seed, dense=False)
        P = _exact_P(c, d, c["warm"] + c["steps"])
        return torch.linalg.solve(_t(d["R"]), _t(d["B"]).t() @ P).cpu().numpy()
    if what == "serve":
        return [_exact_P(r, d, r["steps"]) for r, d in _requests(c, seed)]
    if what == "expm":
        X = _expm_operator(c, seed).t() * c["t"]
        return torch.linalg.matrix_exp(X)
    if what == "expmv":
        gen = torch.Generator("cuda").manual_seed(seed)
        X = torch.randn(c["cols"], c["nx"] ** 2, generator=gen, dtype=torch.float64, device="cuda").t().contiguous()
        return _Grid(c["nx"]).apply(c["t"], X)
    f = _factors(c, seed)
    if what == "riccati":
        W = f["L"].t() @ f["B"]
        G = f["D"] @ W
        return f["D"] - c["t"] * G @ torch.linalg.solve(f["R"] + c["t"] * W.t() @ G, G.t())
    Q, T = torch.linalg.qr(f["W"].cpu())
    lam, V = torch.linalg.eigh(T @ f["D"].cpu() @ T.t())
    keep = lam.abs() > c["tol"] * lam.abs().max()
    X = (Q @ V[:, keep]).cuda()
    return (X * lam[keep].cuda()) @ X.t()
