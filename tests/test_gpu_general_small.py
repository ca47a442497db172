"""The batched kernel of 256 threads for small instances with a non-diagonal Q
(at most 256 variables and rows) and its limits, against the general batched
kernel, with the tolerance of test_gpu_general_batch.py; and more instances
than the chip holds at a time, each with the bits of a batch of its own."""

import numpy as np
import pytest

import paper_2602_23967_amd as P
from test_gpu_general_batch import GENERAL_KERNEL, _qp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need the MI355X"
    return T


@pytest.mark.parametrize("n, m, q_row, a_row", [
    (2, 0, 0, 1), (2, 256, 0, 2), (64, 1, 63, 64), (65, 64, 40, 9), (128, 256, 34, 30), (255, 255, 9, 5), (256, 256, 11, 9),
    (256, 128, 24, 20),     # A past the LDS that Q leaves
    (256, 100, 33, 5),      # Q past a quarter of the LDS: a whole CU
    (256, 257, 9, 5), (224, 257, 9, 5),   # more rows than threads: a whole CU
    (223, 257, 9, 5), (257, 100, 9, 5)])  # the general kernel; a whole CU
def test_small_instances(torch, n, m, q_row, a_row):
    print(n, m, q_row, a_row, flush=True)
    qs = [_qp(n, m, q_row, a_row, s) for s in range(3)]
    kw = dict(max_iter=70, check_every=7, tol=1e-13)
    with P.BatchSolver(qs) as bs:
        got = {}
        for shape in (GENERAL_KERNEL, P.qp_batch_default_shape(False)):
            bs.set_schedule(shape=shape)
            bs.solve(**kw)
            got[shape] = [bs.result(i) for i in range(len(qs))]
    for g, r in zip(got[P.qp_batch_default_shape(False)], got[GENERAL_KERNEL]):
        assert g.status == r.status and g.info["iterations"] == r.info["iterations"]
        assert np.abs(g.x - r.x).max() <= 1e-9 * (1.0 + np.abs(r.x).max())
        if m:
            assert np.abs(g.y - r.y).max() <= 1e-9 * (1.0 + np.abs(r.y).max())


def test_both_workgroups_make_the_same_bits(torch):
    """Alone they take 256 threads; beside a larger instance 1024."""
    qs = [_qp(n, m, q, a, 5) for n, m, q, a in
          [(2, 1, 0, 1), (64, 64, 63, 9), (65, 0, 20, 1), (128, 256, 34, 30), (255, 255, 9, 5), (256, 128, 24, 20)]]
    for kw in (dict(max_iter=70, check_every=7, tol=1e-13), dict(tol=1e-7)):
        got = []
        for extra in ([], [_qp(400, 100, 9, 5, 6)]):
            with P.BatchSolver(qs + extra) as bs:
                bs.solve(**kw)
                got.append([bs.result(i) for i in range(len(qs))])
        for q, a, b in zip(qs, *got):
            assert a.status == b.status, q.name
            for k in ("iterations", "inner_iterations", "restarts", "omega", "r_primal", "r_dual", "primal_obj"):
                assert a.info[k] == b.info[k], (q.name, k)
            assert np.array_equal(a.x, b.x) and np.array_equal(a.y, b.y), q.name


def test_more_instances_than_the_chip_holds(torch):
    kinds = [_qp(n, m, 5, 3, 7) for n, m in [(20, 10), (100, 40), (250, 120)]]
    kw = dict(max_iter=70, check_every=7, tol=1e-13)
    alone = []
    for q in kinds:
        with P.BatchSolver([q]) as bs:
            bs.solve(**kw)
            alone.append(bs.result(0))
    count = 2600
    print(count, "instances", flush=True)
    with P.BatchSolver([kinds[i % 3] for i in range(count)]) as bs:
        bs.solve(**kw)
        for i in range(count):
            r = bs.result(i)
            assert np.array_equal(r.x, alone[i % 3].x) and np.array_equal(r.y, alone[i % 3].y), i
