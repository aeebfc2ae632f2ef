"""Vectors of 4097 to 6144 entries as one chunk: an Arnoldi step, the restart tail and the end of a
cycle in one launch each, with 24 entries per thread.  Alone (the fused launches) and beside a larger
instance in a batch (the launch chains) an instance gives the same bits; the solution is the
oracle's."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1305_6653_amd import BvmSolver, factor_batch, solve_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,s", [(65, 64), (96, 64), (383, 16)])
@pytest.mark.parametrize("restart", [3, 20])
def test_fused_and_chained_steps_agree(m, s, restart):
    p, big = W.tiny(m, s, 1.6, 4, "gbdf3"), W.tiny(200, 64, 1.8, 4, "gbdf3")
    S = BvmSolver(p)
    S.factor("fp64")
    S.profile(True)
    u, info = S.solve(p.u0, p.f, restart=restart)
    assert info["converged"] == 1 and S.profile_query("arnoldi")["count"] == info["iters"]
    assert S.profile_query("mgs")["count"] == 0
    S.profile(False)
    B = [BvmSolver(p), BvmSolver(big)]
    factor_batch(B, "fp64")
    outs, infos = solve_batch(B, [p.u0, big.u0], [p.f, big.f], restart=restart)
    assert np.array_equal(outs[0], u) and infos[0]["iters"] == info["iters"]
    ref = O.solve_gmres(p, tol=1e-12).x
    assert np.linalg.norm(u - ref) <= 1e-9 * np.linalg.norm(ref)
    for T in [S] + B:
        T.close()


def test_first_size_above_keeps_the_chain():
    p = W.tiny(97, 64, 1.6, 4, "gbdf3")
    S = BvmSolver(p)
    S.factor("fp64")
    S.profile(True)
    _, info = S.solve(p.u0, p.f)
    assert S.profile_query("arnoldi")["count"] == 0
    assert S.profile_query("mgs")["count"] == sum(j + 2 for j in range(info["iters"]))
    S.close()
