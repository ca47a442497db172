"""The one-launch iterations with fewer workgroups than slices, as when other
streams hold the CUs: each takes several slices of Q and of A in a round and
the launches are shorter, and the results are the full group's to the bit."""

import ctypes as C

import numpy as np
import pytest

import paper_2602_23967_amd as P
from test_gpu_coop import _qp
from test_gpu_coop_rounds import _subproblem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need the MI355X"
    return T


def _group(s, cap):
    f = P.lib().qp_internal_group
    f.restype, f.argtypes = C.c_int, [C.c_void_p, C.c_int32]
    return f(s.h, cap)


@pytest.mark.parametrize("n, m", [(3000, 0), (3000, 1500), (1100, 9000), (10000, 70000), (40000, 9000)])
def test_any_number_of_workgroups(torch, n, m):
    q = _qp(n, m)
    kw = dict(tol=1e-13, max_iter=70)
    with P.Solver(q) as s:
        full = _group(s, 0)
        assert full > 1
        ref = s.solve(**kw)
        steps, xs, _ = _subproblem(torch, s, q)
        for cap in (1, 2, full // 2, full - 1):
            if cap < 1 or cap * 40 < full:   # one workgroup of a large group: seconds
                continue
            print(n, m, cap, "of", full, flush=True)
            assert _group(s, cap) == full
            got = s.solve(**kw)
            assert got.status == ref.status and got.info["iterations"] == ref.info["iterations"]
            assert got.info["inner_iterations"] == ref.info["inner_iterations"]
            assert np.array_equal(got.x, ref.x) and np.array_equal(got.y, ref.y)
            some, xg, _ = _subproblem(torch, s, q)
            assert some == steps and np.array_equal(xg, xs)
        _group(s, 0)
        again = s.solve(**kw)
        assert np.array_equal(again.x, ref.x) and np.array_equal(again.y, ref.y)
