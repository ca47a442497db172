"""Results of a batch fetched in any order are the same: those fetched in the
instances' order come from the device in blocks of instances, others alone."""

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


def _unbounded():
    """A free variable that no row touches, with a negative cost."""
    q = I.tiny_lp(40)
    A = q.A.toarray()
    A[:, 0] = 0.0
    q.A = sp.csr_matrix(A)
    q.lb = q.lb.copy(); q.ub = q.ub.copy()
    q.lb[0], q.ub[0] = -np.inf, np.inf
    q.c = q.c.copy(); q.c[0] = -1.0
    q.b = q.A @ np.full(q.n, 1.0)
    return q


@pytest.mark.parametrize("count", [1, 2, 3, 1100])   # 1100: more than one block (2 MiB) of results
def test_results_in_any_order(torch, count):
    kinds = [I.mpc(0), I.mpc(100, infeasible=True), _unbounded(), I.tiny_lp(3)]
    print(f"{count} instances", flush=True)
    with P.BatchSolver([kinds[i % 4] for i in range(count)]) as b:
        for iters in (64, 20000):   # the second solve's results replace the first's
            b.solve(max_iter=iters)
            walk = [b.result(i) for i in range(count)]
            back = [b.result(i) for i in reversed(range(count))][::-1]
            skip = {i: b.result(i) for i in range(0, count, 7)}
            late = [b.result(i) for i in range(count // 2, count)]
            for i in range(count):
                for other in [back[i]] + ([skip[i]] if i in skip else []) + ([late[i - count // 2]] if i >= count // 2 else []):
                    assert other.status == walk[i].status
                    assert np.array_equal(other.x, walk[i].x) and np.array_equal(other.y, walk[i].y)
                assert np.array_equal(walk[i].x, walk[i % 4].x) and np.array_equal(walk[i].y, walk[i % 4].y)
        if count >= 3:
            assert walk[1].status == P.PRIMAL_INFEASIBLE and walk[2].status == P.DUAL_INFEASIBLE
