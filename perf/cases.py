"""The work that users of this solver have it do, as cases that can be timed.

listed() holds one case for each way the library is used in earnest, over the
range of sizes of the repository's workloads; draw() gives further cases of
the same ranges.  prepare() makes what a program has in hand before the call
(the problem, its handle or batch, the point it starts from), run() makes one
call through the public binding and returns its whole result.

Kinds:
  apply       one product with Q, A or A' on device buffers (a program with an
              outer method of its own, over the library's operators)
  kkt         the KKT residuals of a given point (checking someone's solution)
  subproblem  one proximal subproblem, the inner conjugate-gradient solve
  general     a solve with a sparse non-diagonal Q (random QP family)
  large       the same for the diagonally dominant family of up to 1e6 variables
  portfolio   a solve with a diagonal Q (factor-model portfolio)
  factored    a solve with Q = P + R'R given by its factors
  mpc         a batch of linear MPC problems, created once and solved
  static      a batch from host arrays to host results in one call
  batch       a batch of small QPs with non-diagonal Q
Solves run to the tolerance (iters 0), for a fixed budget of iterations, as a
program with a deadline runs them, or to whichever comes first.
"""

import numpy as np
import scipy.sparse as sp
import torch

import paper_2602_23967_amd as P
from paper_2602_23967_amd import instances as I


def listed():
    return [
        # the smallest call: one product of a small problem, all latency
        {"name": "apply_at_n1000", "kind": "apply", "op": "AT", "family": "general", "n": 1000},
        # residuals of a point on a large problem, odd size
        {"name": "kkt_n299993", "kind": "kkt", "n": 299993},
        # one inner solve on a large problem, odd size
        {"name": "subproblem_n200003", "kind": "subproblem", "n": 200003},
        # a solve of the tiny random QP to its tolerance (or 2048 iterations), bound by latency
        {"name": "general_n1000", "kind": "general", "n": 1000, "iters": 2048, "tol": 1e-6, "mixed": False},
        # the random QPs of a served stream (n up to 5e4), under a budget
        {"name": "general_n20011", "kind": "general", "n": 20011, "iters": 128, "mixed": False},
        # the large sparse QP of the benchmark, under a budget
        {"name": "large_n1000000", "kind": "large", "n": 1000000, "iters": 64, "mixed": False},
        # the factor portfolio of the benchmark, in the precision it is run in
        {"name": "portfolio_n200000", "kind": "portfolio", "n": 200000, "k": 1000, "iters": 1024, "mixed": True},
        # a portfolio of a served stream in double precision, odd size
        {"name": "portfolio_n31337", "kind": "portfolio", "n": 31337, "k": 156, "iters": 1024, "mixed": False},
        # the portfolio with the factors kept in Q
        {"name": "factored_n50000", "kind": "factored", "n": 50000, "k": 250, "iters": 48, "mixed": False},
        # the MPC batch of the benchmark, in the precision it is run in
        {"name": "mpc_4096", "kind": "mpc", "count": 4096, "mixed": True},
        # a control loop's handful of problems, from host arrays to host results
        {"name": "static_8", "kind": "static", "count": 8, "mixed": False},
        # small QPs with an inner solve in one launch (a server's general lane)
        {"name": "batch_general_24", "kind": "batch", "count": 24, "nmin": 200, "nmax": 1000, "iters": 320,
         "mixed": False},
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["apply", "kkt", "subproblem", "general", "general", "large", "portfolio", "portfolio",
                       "factored", "mpc", "static", "batch"])
    mixed = rng.random() < 0.5
    if kind == "apply":
        fam = rng.choice(["general", "large"])
        return {"kind": kind, "op": rng.choice(["Q", "A", "AT"]), "family": fam,
                "n": _log(rng, 1000, 50000) if fam == "general" else _log(rng, 50000, 1000000)}
    if kind in ("kkt", "subproblem"):
        return {"kind": kind, "n": _log(rng, 20000, 600000)}
    if kind == "general":
        return {"kind": kind, "n": _log(rng, 1000, 50000), "iters": rng.randint(64, 128), "mixed": mixed}
    if kind == "large":
        return {"kind": kind, "n": _log(rng, 50000, 1000000), "iters": rng.randint(32, 64), "mixed": mixed}
    if kind == "portfolio":
        n = _log(rng, 10000, 200000)
        return {"kind": kind, "n": n, "k": max(1, n // 200), "iters": rng.randint(256, 1024), "mixed": mixed}
    if kind == "factored":
        n = _log(rng, 10000, 50000)
        return {"kind": kind, "n": n, "k": max(1, n // 200), "iters": rng.randint(24, 48), "mixed": mixed}
    if kind == "mpc":
        return {"kind": kind, "count": _log(rng, 16, 4096), "mixed": mixed}
    if kind == "static":
        return {"kind": kind, "count": _log(rng, 1, 64), "mixed": mixed}
    nmin = rng.randint(100, 400)
    return {"kind": "batch", "count": rng.randint(4, 48), "nmin": nmin, "nmax": nmin + rng.randint(1, 600),
            "iters": rng.randint(128, 320), "mixed": mixed}


# ---- problems ---------------------------------------------------------------------

def _large(seed, n):
    """The large sparse family (instances.large_sparse) drawn the same way,
    sorted on the GPU: about 10 off-diagonals per row, a dominant diagonal, 8
    entries per row of A, half '=' and half '>=' rows, box [0, 10]."""
    rng = np.random.default_rng([260223967, 1, seed])
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    m = n // 2
    i = rng.integers(0, n, size=5 * n)
    j = rng.integers(0, n - 1, size=5 * n)
    j = j + (j >= i)
    key = torch.unique(torch.from_numpy(np.minimum(i, j) * n + np.maximum(i, j)).to(dev))
    lo, hi = key // n, key % n
    v = torch.from_numpy(rng.normal(size=key.numel())).to(dev)
    both, at = torch.sort(torch.cat([lo * n + hi, hi * n + lo]))
    rows = (both // n).cpu().numpy()
    vals = torch.cat([v, v])[at].cpu().numpy()
    diag = np.bincount(rows, weights=np.abs(vals), minlength=n) + 0.1
    d = torch.arange(n, device=dev)
    full, at = torch.sort(torch.cat([both, d * n + d]))
    qv = torch.cat([torch.from_numpy(vals).to(dev), torch.from_numpy(diag).to(dev)])[at].cpu().numpy()
    qj = (full % n).to(torch.int32).cpu().numpy()
    qp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=n) + 1, out=qp[1:])
    Q = sp.csr_matrix((qv, qj, qp), shape=(n, n))

    cols = np.sort(rng.integers(0, n, size=(m, 8)), axis=1)
    while True:
        bad = np.nonzero((cols[:, 1:] == cols[:, :-1]).any(axis=1))[0]
        if bad.size == 0:
            break
        cols[bad] = np.sort(rng.integers(0, n, size=(bad.size, 8)), axis=1)
    A = sp.csr_matrix((rng.normal(size=8 * m), cols.ravel().astype(np.int32), np.arange(m + 1, dtype=np.int64) * 8),
                      shape=(m, n))
    x0 = rng.uniform(0.0, 5.0, size=n)
    sense = b"E" * (m // 2) + b"G" * (m - m // 2)
    return I.QP(n=n, m=m, Q=Q, A=A, c=rng.normal(size=n), b=A @ x0, sense=sense, lb=np.zeros(n),
                ub=np.full(n, 10.0), name=f"large_{n}")


def _general(seed, n):
    return I.random_small(seed, n=n)


def _mpc_batch(seed, count):
    """`count` MPC problems (instances.mpc: horizon 10 to 50, 12 states, 4
    inputs; one in 64 infeasible) packed block-diagonally, written down
    without a Python loop over rows."""
    rng = np.random.default_rng([260223967, 3, seed])
    ns, nu = 12, 4
    step = ns + nu
    T = np.random.default_rng([260223967, 4, count]).integers(10, 51, size=count)   # the same sizes for every seed
    U, _ = np.linalg.qr(rng.normal(size=(count, ns, ns)))
    lam = rng.uniform(-0.95, 0.95, size=(count, ns))
    lam *= 0.95 / np.abs(lam).max(axis=1, keepdims=True)
    Ad = (U * lam[:, None, :]) @ U.transpose(0, 2, 1)
    Bd = rng.normal(0.0, 0.3, size=(count, ns, nu))
    xinit = rng.uniform(-1.0, 1.0, size=(count, ns))
    xinit[63::64, 0] = 6.0
    voff = np.concatenate([[0], np.cumsum(step * T + ns)]).astype(np.int64)
    roff = np.concatenate([[0], np.cumsum(ns * T + ns)]).astype(np.int64)
    jp, jj, jv, cost, ulim, rhs = [], [], [], [], [], []
    for b in range(count):
        t = int(T[b])
        base = (np.arange(t) * step)[:, None, None] + voff[b]
        # row of step t: x_t (12 columns), u_t (4), x_{t+1} (1), in column order
        col = np.empty((t, ns, step + 1), dtype=np.int32)
        col[:, :, :step] = base + np.arange(step)[None, None, :]
        col[:, :, step] = base[:, :, 0] + step + np.arange(ns)[None, :]
        val = np.empty((t, ns, step + 1))
        val[:, :, :ns] = -Ad[b]
        val[:, :, ns:step] = -Bd[b]
        val[:, :, step] = 1.0
        jj += [np.arange(voff[b], voff[b] + ns, dtype=np.int32), col.ravel()]
        jv += [np.ones(ns), val.ravel()]
        jp += [np.ones(ns, dtype=np.int64), np.full(ns * t, step + 1, dtype=np.int64)]
        cost += [np.tile(np.concatenate([np.ones(ns), np.full(nu, 0.1)]), t), np.ones(ns)]
        ulim += [np.tile(np.concatenate([np.full(ns, 5.0), np.ones(nu)]), t), np.full(ns, 5.0)]
        rhs += [xinit[b], np.zeros(ns * t)]
    n, m = int(voff[-1]), int(roff[-1])
    rp = np.concatenate([[0], np.cumsum(np.concatenate(jp))])
    A = sp.csr_matrix((np.concatenate(jv), np.concatenate(jj), rp), shape=(m, n))
    Q = sp.csr_matrix((np.concatenate(cost), np.arange(n, dtype=np.int32), np.arange(n + 1)), shape=(n, n))
    ub = np.concatenate(ulim)
    return {"count": count, "voff": voff, "roff": roff, "Q": Q, "A": A, "c": np.zeros(n), "b": np.concatenate(rhs),
            "sense": b"E" * m, "lb": -ub, "ub": ub}


def _general_batch(seed, case):
    rng = np.random.default_rng([260223967, 5, case["count"]])                      # the same sizes for every seed
    sizes = rng.integers(case["nmin"], case["nmax"] + 1, size=case["count"])
    return [I.random_small(seed * 64 + i, n=int(s)) for i, s in enumerate(sizes)]


class _Batch:
    """Owns a batch handle."""

    def __init__(self, d):
        self.d = d
        self.h = P.qp_batch_create(d["count"], d["voff"], d["roff"], d["Q"], d["A"], d["c"], d["b"], d["sense"],
                                   d["lb"], d["ub"])

    def __del__(self):
        P.qp_batch_destroy(self.h)


def _params(case):
    kw = {"precision": P.PRECISION_MIXED if case.get("mixed") else P.PRECISION_FP64}
    if case.get("iters"):
        # a budget alone: the tolerance is one that it does not reach
        kw.update(max_iter=case["iters"], tol=case.get("tol", 1e-12))
    return P.qp_params_default(**kw)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


_OPS = {"Q": P.OP_Q, "A": P.OP_A, "AT": P.OP_AT}


def _point(case, seed):
    """The host data of an operator call: the problem and its arguments."""
    kind = case["kind"]
    rng = np.random.default_rng([260223967, 7, seed])
    if kind == "apply":
        q = _general(seed, case["n"]) if case["family"] == "general" else _large(seed, case["n"])
        return q, {"v": rng.normal(size=q.m if case["op"] == "AT" else q.n)}
    q = _large(seed, case["n"])
    if kind == "kkt":
        y = rng.normal(size=q.m)
        y[q.m // 2:] = -np.abs(y[q.m // 2:])        # '>=' rows have y <= 0
        return q, {"x": rng.uniform(0.0, 10.0, size=q.n), "y": y}
    # the subproblem of an outer step: tau of the size that the weight gives
    # (eta of a matrix of norm about 5), rhs = x / tau - c - A'y
    tau = 0.2
    x = np.clip(rng.normal(1.0, 2.0, size=q.n), 0.0, 10.0)
    return q, {"x": x, "tau": tau, "rhs": x / tau - q.c - q.A.T @ rng.normal(size=q.m)}


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("apply", "kkt", "subproblem"):
        q, a = _point(case, seed)
        s = {"kind": kind, "solver": P.Solver(q), "args": {k: _dev(v) if isinstance(v, np.ndarray) else v
                                                           for k, v in a.items()}}
        if kind == "apply":
            s["op"] = _OPS[case["op"]]
            s["out"] = torch.empty(q.m if case["op"] == "A" else q.n, dtype=torch.float64, device="cuda")
        if kind == "subproblem":
            s["start"] = s["args"]["x"].clone()
        return s
    if kind in ("mpc", "static"):
        d = _mpc_batch(seed, case["count"])
        return {"kind": kind, "params": _params(case), **({"batch": _Batch(d)} if kind == "mpc" else {"data": d})}
    if kind == "batch":
        b = P.BatchSolver(_general_batch(seed, case))
        b.set_schedule(shape=P.qp_batch_default_shape(True))
        return {"kind": kind, "params": _params(case), "solver": b}
    if kind == "general":
        q = _general(seed, case["n"])
    elif kind == "large":
        q = _large(seed, case["n"])
    elif kind == "portfolio":
        q = I.portfolio(seed, n_assets=case["n"], k_factors=case["k"])
    else:
        q = I.portfolio_factored(seed, n_assets=case["n"], k_factors=case["k"])
    return {"kind": kind, "params": _params(case), "solver": P.Solver(q)}


def run(state):
    kind = state["kind"]
    if kind == "apply":
        P.qp_apply(state["solver"].h, state["op"], state["args"]["v"], state["out"])
        return state["out"]
    if kind == "kkt":
        return P.qp_kkt(state["solver"].h, state["args"]["x"], state["args"]["y"])
    if kind == "subproblem":
        x = state["args"]["x"]
        x.copy_(state["start"])
        torch.cuda.current_stream().synchronize()   # the call runs on the handle's own stream
        it, res = P.qp_subproblem(state["solver"].h, state["args"]["tau"], state["args"]["rhs"], x, 1e-6)
        return {"x": x, "iters": it, "res": res}
    if kind == "static":
        d = state["data"]
        _, x, y, status, _ = P.qp_batch_solve_static(d["count"], d["voff"], d["roff"], d["Q"], d["A"], d["c"], d["b"],
                                                     d["sense"], d["lb"], d["ub"], state["params"])
        return {"x": x, "y": y, "status": status}
    if kind == "mpc":
        d, h = state["batch"].d, state["batch"].h
        P.qp_batch_solve(h, state["params"])
        got = [P.qp_batch_result(h, i, int(d["voff"][i + 1] - d["voff"][i]), int(d["roff"][i + 1] - d["roff"][i]))
               for i in range(d["count"])]
        return {"x": np.concatenate([g[1] for g in got]), "y": np.concatenate([g[2] for g in got]),
                "status": np.array([g[0] for g in got], dtype=np.int32)}
    if kind == "batch":
        b = state["solver"]
        b.solve(state["params"])
        got = [b.result(i) for i in range(len(b.qps))]
        return {"x": np.concatenate([g.x for g in got]), "y": np.concatenate([g.y for g in got]),
                "status": np.array([g.status for g in got], dtype=np.int32)}
    r = state["solver"].solve(state["params"])
    return {"x": r.x, "y": r.y, "status": r.status, "iterations": r.info["iterations"]}


def _sizes(case):
    """(n, m, nonzeros of Q, nonzeros of A) that the families have on average."""
    kind = case["kind"]
    n = case.get("n", 0)
    if kind == "general" or case.get("family") == "general":
        return n, n // 2, 13.2 * n, 5.0 * n
    if kind in ("large", "kkt", "subproblem", "apply"):
        return n, n // 2, 11.0 * n, 4.0 * n
    if kind == "portfolio":
        return n + case["k"], case["k"] + 1, float(n + case["k"]), 0.01 * n * case["k"] + n + case["k"]
    if kind == "factored":
        return n, 1, n + 0.01 * n * case["k"], float(n)
    c = case["count"]
    if kind in ("mpc", "static"):
        return 492.0 * c, 372.0 * c, 492.0 * c, 6132.0 * c
    n = c * (case["nmin"] + case["nmax"]) / 2.0
    return n, n / 2, 13.2 * n, 5.0 * n


def work(case):
    """One pass: the problem and the start read once, the result written once;
    the arithmetic of the iterations that it makes (8 inner steps in each with
    a non-diagonal Q; about 3000 iterations for MPC solved to its tolerance)."""
    n, m, nq, na = _sizes(case)
    kind = case["kind"]
    if kind == "apply":
        nnz = nq if case["op"] == "Q" else na
        rows = m if case["op"] == "A" else n
        cols = m if case["op"] == "AT" else n
        return {"bytes": 12.0 * nnz + 4 * (rows + 1) + 8 * rows + 8 * cols, "flops": 2.0 * nnz}
    read = 12.0 * (nq + na) + 4 * (n + m + 2) + 8 * (3 * n + 2 * m)
    if kind == "kkt":
        return {"bytes": read + 8 * (n + m), "flops": 2.0 * (nq + 2 * na) + 10 * (n + m)}
    if kind == "subproblem":
        return {"bytes": 12.0 * nq + 4 * (n + 1) + 8 * 3 * n, "flops": 12 * (2.0 * nq + 20 * n)}
    iters = case.get("iters") or 3000
    inner = 8 if kind in ("general", "large", "factored", "batch") else 0
    per = 4.0 * na + 15 * (n + m) + inner * (2.0 * nq + 20 * n)
    return {"bytes": read + 8 * (n + m), "flops": iters * per}


# ---- the results in 64 bits, by numpy and scipy ------------------------------------

def _exact_kkt(q, x, y):
    inf = np.inf
    l, u = q.lb, q.ub
    lc = q.b
    uc = np.where(np.frombuffer(q.sense, dtype=np.uint8) == ord("E"), q.b, inf)
    Qx, Aty, Ax = q.Q @ x, q.A.T @ y, q.A @ x
    r = Qx + q.c + Aty
    fin = np.isfinite(uc)

    def support(z, lo, hi):
        return np.sum(np.where(z > 0, np.where(z > 0, hi, 0.0) * z, np.where(z < 0, lo * z, 0.0)))

    with np.errstate(invalid="ignore"):
        pr = support(-r, l, u)                       # every variable is boxed: proj_R is the identity
        py = support(y, lc, uc)
    pviol = np.max(np.abs(Ax - np.clip(Ax, lc, uc)))
    xqx, cx = x @ Qx, q.c @ x
    pobj, dneg = 0.5 * xqx + cx, 0.5 * xqx + pr + py
    bnd = max(np.max(np.abs(lc)), np.max(np.abs(uc[fin])))
    return {"r_primal": float(pviol / (1 + bnd)), "r_dual": 0.0,
            "r_gap": float(abs(xqx + cx + pr + py) / (1 + max(abs(pobj), abs(dneg)))),
            "pobj": float(pobj), "dobj": float(-dneg),
            "natural": float(np.max(np.abs(x - np.clip(x - r, l, u)))), "pviol": float(pviol)}


def _exact_box_qp(q, tau, rhs, x0):
    """argmin over the box of 1/2 x'(Q + I/tau)x - rhs'x by the primal-dual
    active set method, the free block solved by scipy's conjugate gradients."""
    from scipy.sparse.linalg import cg
    H = (q.Q + sp.identity(q.n, format="csr") / tau).tocsr()
    x, diag = x0.copy(), H.diagonal()
    lo = up = None
    for _ in range(60):
        z = x - (H @ x - rhs) / diag
        lo2, up2 = z <= q.lb, z >= q.ub
        if lo is not None and np.array_equal(lo, lo2) and np.array_equal(up, up2):
            return x
        lo, up = lo2, up2
        x = np.where(lo, q.lb, np.where(up, q.ub, x))
        f = np.nonzero(~(lo | up))[0]
        fixed = np.where(lo | up, x, 0.0)
        Hf = H[f][:, f]
        x[f], info = cg(Hf, (rhs - H @ fixed)[f], x0=x[f], rtol=1e-14, maxiter=400,
                        M=sp.diags(1.0 / diag[f]))
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("apply", "kkt", "subproblem"):
        return None          # iterates of a method, not a number that another method has
    q, a = _point(case, seed)
    if kind == "apply":
        return {"Q": q.Q, "A": q.A, "AT": q.A.T}[case["op"]] @ a["v"]
    if kind == "kkt":
        return _exact_kkt(q, a["x"], a["y"])
    return {"x": _exact_box_qp(q, a["tau"], a["rhs"], a["x"]), "iters": None, "res": None}
