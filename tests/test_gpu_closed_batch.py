"""The batched kernels that keep a whole instance on one CU (diagonal Q, at
most 1024 variables and rows): sizes at the edges of their tiles, rows longer
than their registers and their LDS hold, against the oracle's iterates."""

import numpy as np
import pytest
import scipy.sparse as sp

import oracle
import paper_2602_23967_amd as P
from paper_2602_23967_amd import instances as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need the MI355X"
    return T


def _diag_qp(n, m, per_row, seed):
    """Diagonal Q, m rows of per_row entries each, a box and mixed senses."""
    rng = np.random.default_rng([9, n, m, seed])
    k = min(per_row, n)
    cols = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for _ in range(m)]) if m else np.zeros(0, int)
    A = sp.csr_matrix((rng.normal(size=m * k), cols, np.arange(m + 1) * k), shape=(m, n))
    x0 = rng.uniform(-0.5, 0.5, size=n)
    sense = b"".join(b"EGL"[i % 3:i % 3 + 1] for i in range(m))
    slack = np.array([0.0, -0.1, 0.1])[np.arange(m) % 3]
    return I.QP(n=n, m=m, Q=sp.diags(rng.uniform(0.1, 1.0, size=n)).tocsr(), A=A, c=rng.normal(size=n), b=A @ x0 + slack,
                sense=sense, lb=np.full(n, -1.0), ub=np.where(np.arange(n) % 5 == 0, np.inf, 1.0), name=f"diag_{n}_{m}_{k}")


@pytest.mark.parametrize("n, m, per_row", [
    (1, 1, 1), (63, 1, 63), (64, 64, 5), (65, 63, 17), (257, 129, 33),
    (1024, 5, 256),      # one wave's rows alone longer than LDS holds of them
    (1023, 1024, 4), (1024, 1024, 24),   # A past the LDS: the last waves' rows from memory
    (130, 250, 130),     # columns of up to 250 entries: past the registers
    (1025, 7, 9), (40, 1025, 3)])        # just too large: the general batched kernel
def test_closed_instances_match_oracle(torch, n, m, per_row):
    """Iterates after 70 iterations (checks every 7) equal the oracle's up to
    the order of their sums; the mixed solve's result meets the tolerance."""
    qs = [_diag_qp(n, m, per_row, s) for s in range(2)]
    with P.BatchSolver(qs) as bs:
        bs.solve(max_iter=70, check_every=7, tol=1e-13)
        res = [bs.result(i) for i in range(len(qs))]
        for q, g in zip(qs, res):
            o = oracle.solve(q, max_iter=70, check_every=7, tol=1e-13)
            assert g.status == o.status and g.info["iterations"] == o.info["iterations"], q.name
            assert g.info["restarts"] == o.info["restarts"], q.name
            err = max(np.abs(g.x - o.x).max() / (1.0 + np.abs(o.x).max()),
                      np.abs(g.y - o.y).max() / (1.0 + np.abs(o.y).max()))
            assert err <= 1e-10, (q.name, err)
        bs.solve(precision=P.PRECISION_MIXED)
        for i, q in enumerate(qs):
            g = bs.result(i)
            k = oracle.kkt(q, g.x, g.y)
            assert g.status == P.OPTIMAL and max(k["r_primal"], k["r_dual"], k["r_gap"]) <= 1e-6, (q.name, k)


@pytest.mark.parametrize("n, m, per_row", [(65, 63, 17), (1024, 1024, 24), (130, 250, 130)])
def test_closed_norm_matches_svd(torch, n, m, per_row):
    """||A||_2 by power iteration (stopped at a relative change of 1e-7)."""
    q = _diag_qp(n, m, per_row, 0)
    with P.BatchSolver([q]) as bs:
        bs.solve(max_iter=1)
        assert bs.result(0).info["norm_A"] == pytest.approx(np.linalg.norm(q.A.toarray(), 2), rel=1e-3)
