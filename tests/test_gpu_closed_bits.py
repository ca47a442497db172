"""The batched kernels that keep a closed-form instance on one CU make the
general batched kernel's iterates to the bit, in both precisions: the default
shape against one of 256 threads that sends every instance to the general
kernel, through checks, restarts, unbounded variables, certificates and
rows past the registers and the LDS.

The check's own sums (residuals, objectives) are grouped by the workgroup's
size, and the movement that a certificate of primal infeasibility scales is a
difference whose product may be fused: entries of at most 1 with an absolute
error of some 2^-53 * |y| / max|movement|, tested as 1e-12.
"""

import numpy as np
import pytest

import paper_2602_23967_amd as P
from paper_2602_23967_amd import instances as I
from test_gpu_closed_batch import _diag_qp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need the MI355X"
    return T


def _general_shape():
    """A compiled shape of 256 threads (its sums have the same order) that is not a default."""
    for s in range(P.qp_batch_num_shapes()):
        if P.qp_batch_shape_info(s)[0] == 256 and s not in (P.qp_batch_default_shape(False), P.qp_batch_default_shape(True)):
            return s


def _free(q):
    """The same with every third variable unbounded below or above."""
    q.lb = q.lb.copy(); q.ub = q.ub.copy()
    q.lb[::3], q.ub[1::4] = -np.inf, np.inf
    return q


@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
def test_same_bits_as_the_general_kernel(torch, precision):
    qs = [_diag_qp(n, m, k, 3) for n, m, k in
          [(1, 1, 1), (5, 0, 1), (16, 8, 5), (63, 1, 63), (64, 64, 5), (65, 63, 17), (257, 129, 33), (1024, 5, 256),
           (1023, 1024, 4), (1024, 1024, 24), (130, 250, 130)]]
    qs += [_free(_diag_qp(n, m, k, 4)) for n, m, k in [(40, 20, 7), (300, 200, 11), (900, 500, 6)]]
    qs += [I.mpc(i) for i in range(6)] + [I.mpc(100, infeasible=True), I.tiny_lp(3), I.tiny_lp(5, n=90, m=40)]
    other = _general_shape()
    default = P.qp_batch_default_shape(False)
    restarts = 0
    with P.BatchSolver(qs) as bs:
        for kw in (dict(max_iter=70, check_every=7, tol=1e-13), dict(max_iter=1000, check_every=16, tol=1e-13),
                   dict(tol=1e-6), dict(max_iter=70, check_every=7, tol=1e-13, use_halpern=0)):
            got = {}
            for shape in (other, default):
                print("shape", shape, kw, flush=True)
                bs.set_schedule(shape=shape)
                bs.solve(precision=precision, **kw)
                got[shape] = [bs.result(i) for i in range(len(qs))]
            for q, a, b in zip(qs, got[other], got[default]):
                for k in ("iterations", "restarts", "omega"):
                    assert a.info[k] == b.info[k], (q.name, kw, k, a.info[k], b.info[k])
                assert a.status == b.status and np.array_equal(a.x, b.x), (q.name, kw)
                if a.status == P.PRIMAL_INFEASIBLE:
                    assert np.abs(a.y - b.y).max() <= 1e-12, (q.name, kw)
                else:
                    assert np.array_equal(a.y, b.y), (q.name, kw)
                restarts += a.info["restarts"]
    assert restarts > 0
