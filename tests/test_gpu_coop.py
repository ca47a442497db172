"""A non-diagonal Q's iterations in one launch against the launch-by-launch
path, which a solve that times its kernels takes on the same handle.

Both make the same iterations in another order of summation.  Each of K = 130
iterations of about 10 steps adds a relative error of at most some 100 * 2^-53
to iterates that the method does not expand: 130 * 10 * 100 * 1.1e-16 = 1.5e-11,
tested as 1e-9 of the largest entry.  In
mixed precision both are the launch-by-launch path.
"""

import numpy as np
import pytest
import scipy.sparse as sp

import paper_2602_23967_amd as P
from paper_2602_23967_amd import instances as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need the MI355X"
    return T


def _qp(n, m, qrow=4, acol=0, seed=0, unbounded=False):
    """Random QP; row 0 of Q has qrow off-diagonals, column 0 of A acol entries."""
    rng = np.random.default_rng([260223967, 71, n, m, qrow, acol, seed])
    S = sp.random(n, n, density=min(1.0, 3.0 / n), random_state=rng, format="lil")
    S.setdiag(0.0)
    S[0, :] = 0.0
    S[:, 0] = 0.0
    if n > 1:
        k = min(qrow, n - 1)
        S[0, 1:1 + k] = rng.normal(size=k)
    S = S.tocsr()
    S.eliminate_zeros()
    S = S + S.T
    Q = (S + sp.diags(np.asarray(abs(S).sum(axis=1)).ravel() + 0.5)).tocsr()
    A = sp.random(m, n, density=min(1.0, 5.0 / n), random_state=rng, format="lil")
    if acol:
        A[:acol, 0] = rng.normal(size=(acol, 1))
    A = A.tocsr()
    x0 = rng.uniform(-0.5, 0.5, size=n)
    lb, ub = np.full(n, -1.0), np.full(n, 1.0)
    if unbounded:
        lb[::3], ub[1::4] = -np.inf, np.inf
    return I.QP(n=n, m=m, Q=Q, A=A, c=rng.normal(size=n), b=A @ x0, sense=b"E" * (m // 2) + b"G" * (m - m // 2),
                lb=lb, ub=ub, name=f"coop_{n}_{m}")


# on one CU: up to 1000 variables; with a group of workgroups: the longest
# rows, more than 1024 variables or rows.  Its row limit (256) met and passed, more rows of A than of Q;
# the longest row and column that the path takes, and one entry more (then both routes are one)
CASES = [dict(n=1, m=1), dict(n=3, m=0), dict(n=255, m=128), dict(n=256, m=300), dict(n=257, m=64),
         dict(n=700, m=2000), dict(n=1000, m=500, qrow=255), dict(n=1000, m=500, qrow=256),
         dict(n=1024, m=1024), dict(n=1025, m=3), dict(n=600, m=400, acol=64), dict(n=600, m=400, acol=65), dict(n=5000, m=2500, unbounded=True),
         dict(n=40000, m=9000)]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(str(v) for v in c.values()))
def test_same_iterates(torch, case, precision):
    print(f"{case} precision {precision}", flush=True)
    q = _qp(**case)
    with P.Solver(q) as s:
        kw = dict(tol=1e-13, max_iter=130, precision=precision)
        ref = s.solve(timing=1, **kw)
        got = s.solve(**kw)
        again = s.solve(**kw)
    assert got.status == ref.status and got.info["iterations"] == ref.info["iterations"]
    tol = 0.0 if precision else 1e-9
    assert np.abs(got.x - ref.x).max() <= tol * max(1.0, np.abs(ref.x).max())
    if q.m:
        assert np.abs(got.y - ref.y).max() <= tol * max(1.0, np.abs(ref.y).max())
    assert np.array_equal(got.x, again.x) and np.array_equal(got.y, again.y)


def test_subproblem(torch):
    q = _qp(3000, 100)
    with P.Solver(q) as s:
        rng = np.random.default_rng(5)
        rhs = torch.from_numpy(rng.normal(size=q.n)).cuda()
        x = torch.zeros(q.n, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        steps, res = P.qp_subproblem(s.h, 0.5, rhs, x, 1e-12, 1000)[:2]
        xs = x.cpu().numpy()
    # optimality of the box-constrained subproblem: the projected gradient vanishes
    g = q.Q @ xs + 2.0 * xs - rhs.cpu().numpy()
    pg = xs - np.clip(xs - g, q.lb, q.ub)
    assert 0 < steps < 1000 and np.abs(pg).max() <= 1e-11
