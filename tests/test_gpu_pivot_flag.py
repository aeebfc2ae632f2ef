"""The pivot flag of a factorization lies in host memory that the kernels write: every route still
reports a singular block, twice in a row, and a factorization that succeeds does not see an older
failure of its batch."""
import types

import numpy as np
import pytest

import workloads as W
from paper_1305_6653_amd import BvmSolver, FdeError, factor_batch
from paper_1305_6653_amd import _native as N

pytestmark = pytest.mark.gpu

# sigma = 0 and a double root of rho at 1: K_0 = rho(1) I = 0
SINGULAR = types.SimpleNamespace(nu=1, mu=2, alpha=[1.0, -2.0, 1.0], beta=[0.0, 0.0, 0.0], alpha_init=[], beta_init=[],
                                 alpha_fin=[1.0, -2.0, 1.0], beta_fin=[0.0, 0.0, 0.0])


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("m,s", [(20, 8), (20, 64), (300, 16)])
@pytest.mark.parametrize("blocks", ["auto", "lu", "hessenberg", "band"])
def test_singular_blocks_are_reported(blocks, m, s, prec):
    p = W.tiny(m, s, 1.5, 9, "gbdf3")
    S, G = BvmSolver(p, formula=SINGULAR), BvmSolver(p)
    for _ in range(2):
        with pytest.raises(FdeError) as e:
            S.factor(prec, blocks=blocks)
        assert e.value.status == N.FDE_ESINGULAR
    G.factor(prec, blocks=blocks)
    with pytest.raises(FdeError) as e:
        factor_batch([S, G], prec)
    assert e.value.status == N.FDE_ESINGULAR
    G.factor(prec, blocks=blocks)
    u, info = G.solve(p.u0, p.f)
    assert info["converged"] == 1 and np.all(np.isfinite(u))
    S.close()
    G.close()
