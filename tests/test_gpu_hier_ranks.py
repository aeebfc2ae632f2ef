"""The first factor kernel of the hierarchical form (leaf inverses, level 0 and the columns of the
levels above) at the ends of its ranges: alpha near 1 (level 0 at its largest rank, 20) and near 2
(ranks below one tile), pairs with a missing second leaf, and numbers of higher-level columns from
none to more than one pass of four tiles.  Blocks as the oracle's LAPACK solves give them."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1305_6653_amd import BvmSolver
from paper_1305_6653_amd import _native as N

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,eps", [("fp64", 2.0 ** -53), ("mixed", 2.0 ** -24)])
@pytest.mark.parametrize("m,alpha", [(63, 1.3), (127, 1.001), (128, 1.999), (129, 1.5), (192, 1.9999),
                                     (250, 1.001), (600, 1.999), (1030, 1.02)])
def test_first_factor_kernel(m, alpha, prec, eps):
    """Forward error of S^{-1} v within 30 eps max_k cond(K_k), the dense route's bound."""
    p = W.random_instance(11, m=m, s=8)
    p.alpha = alpha
    S = BvmSolver(p)
    S.set_option(N.FDE_OPT_COMPRESS, 2)
    S.factor(prec)
    assert S.get_option(N.FDE_OPT_COMPRESS_IN_USE) == 1
    J, F, tau, _ = O.problem_matrices(p)
    P = O.StrangPreconditioner(J, F, p.s, tau)
    kappa = max(np.linalg.cond(P.block(k, J, tau)) for k in range(p.s // 2 + 1))
    v = np.random.default_rng(4).standard_normal((p.s, p.m))
    ref = P.apply(v)
    assert np.linalg.norm(S.precond(v) - ref) <= 30 * eps * max(kappa, 10.0) * np.linalg.norm(ref)
    S.close()
