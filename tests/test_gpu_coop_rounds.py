"""The one-launch iterations where the slices of Q and of A differ in number,
so that some workgroups own rows of one matrix only: no rows of A at all, one
row, more of A than of Q, more slices of A than compute units; and beside
other work on the GPU.

Against the launch-by-launch path, as in test_gpu_coop.py and with its
tolerance.  Repeats and solves beside other work give the same bits.
"""

import numpy as np
import pytest

import paper_2602_23967_amd as P
from test_gpu_coop import _qp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need the MI355X"
    return T


SHAPES = [(3000, 0), (3000, 1), (1025, 0), (1100, 9000), (1500, 4000), (10000, 70000)]


@pytest.mark.parametrize("n, m", SHAPES)
def test_same_iterates(torch, n, m):
    print(n, m, flush=True)
    q = _qp(n, m)
    kw = dict(tol=1e-13, max_iter=130)
    with P.Solver(q) as s:
        ref = s.solve(timing=1, **kw)
        got = s.solve(**kw)
        for _ in range(3):
            again = s.solve(**kw)
            assert np.array_equal(got.x, again.x) and np.array_equal(got.y, again.y)
    assert got.status == ref.status and got.info["iterations"] == ref.info["iterations"]
    assert np.abs(got.x - ref.x).max() <= 1e-9 * max(1.0, np.abs(ref.x).max())
    if m:
        assert np.abs(got.y - ref.y).max() <= 1e-9 * max(1.0, np.abs(ref.y).max())


def _subproblem(torch, s, q):
    rhs = torch.from_numpy(np.random.default_rng(5).normal(size=q.n)).cuda()
    x = torch.zeros(q.n, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    steps = P.qp_subproblem(s.h, 0.5, rhs, x, 1e-12, 1000)[0]
    return steps, x.cpu().numpy(), rhs.cpu().numpy()


@pytest.mark.parametrize("n, m", SHAPES)
def test_subproblem(torch, n, m):
    print(n, m, flush=True)
    q = _qp(n, m)
    with P.Solver(q) as s:
        steps, xs, rhs = _subproblem(torch, s, q)
        again = _subproblem(torch, s, q)[1]
    # optimality of the box-constrained subproblem: the projected gradient vanishes
    pg = xs - np.clip(xs - (q.Q @ xs + 2.0 * xs - rhs), q.lb, q.ub)
    assert 0 < steps < 1000 and np.abs(pg).max() <= 1e-11
    assert np.array_equal(xs, again)


@pytest.mark.parametrize("n, m", [(3000, 0), (20000, 10000), (1100, 9000)])
def test_beside_work_of_another_stream(torch, n, m):
    print(n, m, flush=True)
    q = _qp(n, m)
    side = torch.cuda.Stream()
    with P.Solver(q) as s:
        idle = s.solve(tol=1e-13, max_iter=130)
        a = torch.rand(1 << 24, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(2000):   # some 20 us each: longer than the solve
                a.mul_(0.999)
        busy = s.solve(tol=1e-13, max_iter=130)
        torch.cuda.synchronize()
    assert np.array_equal(idle.x, busy.x) and np.array_equal(idle.y, busy.y)
