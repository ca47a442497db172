"""Batches whose instances go to different kernels: closed form and inner
solve, on one CU or past it.  The kernels run at the same time (the times of
the instances overlap), and every result equals to the bit that of a batch
with instances of its kind alone."""

import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2602_23967_amd as P
from paper_2602_23967_amd import instances as I
from test_gpu_closed_batch import _diag_qp
from test_gpu_general_batch import _qp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need the MI355X"
    return T


KINDS = {
    "closed": lambda s: _diag_qp(200, 100, 5, s),
    "large closed": lambda s: _diag_qp(1500, 700, 5, s),
    "general": lambda s: _qp(500, 250, 9, 5, s),
    "small general": lambda s: _qp(120, 60, 9, 5, s),
    "large general": lambda s: _qp(1300, 500, 9, 5, s),
}
KW = dict(max_iter=150, check_every=25, tol=1e-13)


def _mix(kinds):
    return [(k, KINDS[k](s)) for s in range(3) for k in kinds]


@pytest.mark.parametrize("precision", [P.PRECISION_FP64, P.PRECISION_MIXED])
@pytest.mark.parametrize("general", [False, True])
def test_results_do_not_depend_on_the_mix(torch, general, precision):
    items = _mix(KINDS)
    shape = P.qp_batch_default_shape(general)

    def solve(qs):
        with P.BatchSolver(qs) as bs:
            bs.set_schedule(shape=shape)
            out = []
            for _ in range(2):   # the second launch finds the first one's streams and counters
                bs.solve(precision=precision, **KW)
                out.append([bs.result(i) for i in range(len(qs))])
            for a, b in zip(*out):
                assert np.array_equal(a.x, b.x) and np.array_equal(a.y, b.y)
            return out[0]

    mixed = solve([q for _, q in items])
    for kind in KINDS:
        print(kind, shape, precision, flush=True)
        at = [i for i, (k, _) in enumerate(items) if k == kind]
        for i, r in zip(at, solve([items[i][1] for i in at])):
            assert r.status == mixed[i].status
            assert np.array_equal(r.x, mixed[i].x) and np.array_equal(r.y, mixed[i].y), kind


def test_static_call_with_all_kinds(torch):
    qs = [q for _, q in _mix(KINDS)]
    big, vo, ro = I.pack(qs)
    params = P.qp_params_default(**KW)
    with P.BatchSolver(qs) as bs:
        bs.solve(params)
        ref = [bs.result(i) for i in range(len(qs))]
    for _ in range(2):
        x, y = P.qp_batch_solve_static(len(qs), vo, ro, big.Q, big.A, big.c, big.b, big.sense, big.lb, big.ub, params=params)[1:3]
        for i, r in enumerate(ref):
            assert np.array_equal(x[vo[i]:vo[i + 1]], r.x) and np.array_equal(y[ro[i]:ro[i + 1]], r.y)


def _overlap():
    """Busy time of the kinds over the time of the solve: 1 when they run one after the other."""
    items = _mix(["closed", "large closed", "general"])
    with P.BatchSolver([q for _, q in items]) as bs:
        for _ in range(3):
            bs.solve(max_iter=600, tol=1e-15)
        start, end = bs.times()
    span = {k: (min(start[i] for i, (kk, _) in enumerate(items) if kk == k),
                max(end[i] for i, (kk, _) in enumerate(items) if kk == k)) for k, _ in items}
    print({k: (round(1e3 * s, 3), round(1e3 * e, 3)) for k, (s, e) in span.items()}, flush=True)
    return sum(e - s for s, e in span.values()) / (max(e for _, e in span.values()) - min(s for s, _ in span.values()))


def test_kinds_run_at_the_same_time(torch):
    # in a process of its own: the streams of a process share four hardware queues
    here = os.path.dirname(os.path.abspath(__file__))
    p = subprocess.run([sys.executable, "-c", "import test_gpu_batch_kinds as t; print('overlap', t._overlap())"],
                       capture_output=True, text=True, timeout=100, cwd=here,
                       env=dict(os.environ, PYTHONPATH=os.pathsep.join([os.path.dirname(here), here])))
    print(p.stdout, p.stderr[-2000:], flush=True)
    assert p.returncode == 0 and float(p.stdout.split("overlap")[1]) > 1.3
