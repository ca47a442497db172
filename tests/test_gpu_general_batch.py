"""The batched kernel that keeps an instance with a non-diagonal Q on one CU
(at most 1024 variables and rows) against the general batched kernel, which
another launch shape runs on the same batch: sizes at the edges of its tiles,
rows of Q longer than the registers and the LDS hold, A past the LDS.

Both make the same iterations in another order of summation; 70 iterations of
about 10 steps with relative errors of at most some 100 * 2^-53 each add up to
70 * 10 * 100 * 1.1e-16 = 8e-12, tested as 1e-9.  In mixed precision the
general kernel runs in all shapes, each with its own order of the reductions,
and an operand's last FP64 bit can move its FP32 rounding (6e-8): 1e-5.
"""

import numpy as np
import pytest
import scipy.sparse as sp

import paper_2602_23967_amd as P
from paper_2602_23967_amd import instances as I

pytestmark = pytest.mark.gpu

GENERAL_KERNEL = 1   # a shape whose instances all run in the general kernel


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need the MI355X"
    return T


def _qp(n, m, q_row, a_row, seed):
    """Symmetric Q with about q_row off-diagonals a row (0: only Q_01), m rows of a_row entries."""
    rng = np.random.default_rng([260223967, 72, n, m, q_row, a_row, seed])
    if q_row:
        S = sp.random(n, n, density=min(1.0, q_row / 2.0 / n), random_state=rng, format="csr")
        S = S - sp.diags(S.diagonal())
        S = S + S.T
    else:
        S = sp.csr_matrix(([0.25, 0.25], ([0, 1], [1, 0])), shape=(n, n))
    Q = (S + sp.diags(np.asarray(abs(S).sum(axis=1)).ravel() + 0.3)).tocsr()
    k = min(a_row, n)
    cols = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for _ in range(m)]) if m else np.zeros(0, int)
    A = sp.csr_matrix((rng.normal(size=m * k), cols, np.arange(m + 1) * k), shape=(m, n))
    x0 = rng.uniform(-0.5, 0.5, size=n)
    sense = b"".join(b"EGL"[i % 3:i % 3 + 1] for i in range(m))
    return I.QP(n=n, m=m, Q=Q, A=A, c=rng.normal(size=n), b=A @ x0 + np.array([0.0, -0.1, 0.1])[np.arange(m) % 3],
                sense=sense, lb=np.full(n, -1.0), ub=np.where(np.arange(n) % 5 == 0, np.inf, 1.0),
                name=f"general_{n}_{m}_{q_row}_{a_row}")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n, m, q_row, a_row", [
    (2, 1, 0, 1), (63, 20, 5, 3), (64, 64, 16, 5), (65, 1, 17, 65), (257, 129, 40, 9),
    (200, 100, 199, 20),      # a dense Q: rows past the registers and past the LDS
    (1023, 1024, 11, 24),     # A past the LDS: the last waves' rows from memory
    (1024, 512, 11, 10),
    (1025, 7, 6, 9), (40, 1025, 6, 3)])   # just too large: the general kernel in both
def test_general_instances(torch, n, m, q_row, a_row, precision):
    print(n, m, q_row, a_row, precision, flush=True)
    qs = [_qp(n, m, q_row, a_row, s) for s in range(2)] + [I.mpc(0)]
    kw = dict(max_iter=70, check_every=7, tol=1e-13, precision=precision)
    with P.BatchSolver(qs) as bs:
        got = {}
        for shape in (GENERAL_KERNEL, P.qp_batch_default_shape(True), P.qp_batch_default_shape(False)):
            bs.set_schedule(shape=shape)
            bs.solve(**kw)
            got[shape] = [bs.result(i) for i in range(2)]
    ref = got.pop(GENERAL_KERNEL)
    tol = 1e-5 if precision else 1e-9
    for res in got.values():
        for g, r in zip(res, ref):
            assert g.status == r.status and g.info["iterations"] == r.info["iterations"]
            assert np.abs(g.x - r.x).max() <= tol * (1.0 + np.abs(r.x).max())
            assert np.abs(g.y - r.y).max() <= tol * (1.0 + np.abs(r.y).max())
