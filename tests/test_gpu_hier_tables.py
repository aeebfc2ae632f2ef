"""The basis tables of the hierarchical form depend on alpha alone: they are built when a factorization
takes the form, not at set-up or with new coefficients, and again only for another alpha."""
import time

import numpy as np
import pytest

import workloads as W
from paper_1305_6653_amd import BvmSolver
from paper_1305_6653_amd import _native as N

pytestmark = pytest.mark.gpu


def test_coefficients_alone_do_not_pay_for_the_tables():
    """4095 rows: the tables take more than 2 ms of the host, the rest of the call a fraction of one."""
    p = W.tiny(4095, 4, 1.4, 2, "gbdf3")
    S = BvmSolver(p)
    took = []
    for i in range(20):
        t = time.perf_counter()
        S.set_coefficients(p.alpha, p.d_plus * (1.0 + 0.01 * i), p.d_minus)
        took.append(time.perf_counter() - t)
    assert min(took) < 1.2e-3, min(took)
    S.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_tables_follow_alpha(prec):
    """Old alpha, another one, back again, with and without a factorization in between: every time the
    bits of a handle that is new."""
    base = W.tiny(700, 8, 1.3, 4, "gbdf3")
    v = np.random.default_rng(8).standard_normal((base.s, base.m))
    S = BvmSolver(base)
    for alpha, factor in ((1.3, True), (1.3, True), (1.7, True), (1.3, False), (1.7, True), (1.05, False), (1.3, True)):
        q = W.tiny(700, 8, alpha, 5, "gbdf3")
        S.set_coefficients(alpha, q.d_plus, q.d_minus)
        if not factor:
            continue
        S.factor(prec)
        assert S.get_option(N.FDE_OPT_COMPRESS_IN_USE) == 1
        T = BvmSolver(q)
        T.factor(prec)
        assert np.array_equal(S.precond(v), T.precond(v)), alpha
        T.close()
    S.close()
