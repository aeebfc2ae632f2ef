"""Modified Gram-Schmidt in two passes over the basis (vectors of more than 7168 entries) at its
edges: the smallest vectors that take it, ragged last chunks, the chunk limit, more than 16 basis
vectors (two groups per pass), restarts, left preconditioning, and batches that mix it with the
launch chain and with one-chunk instances.  Solutions against the oracle, iteration counts against
the classical Gram-Schmidt (twice) of the same system, batches against single solves bit for bit."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1305_6653_amd import BvmSolver, factor_batch, solve_batch
from paper_1305_6653_amd import _native as N

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b))


CASES = {
    "n7176": (lambda: W.tiny(897, 8, 1.5, 1, "gbdf3"), 20),       # 15 chunks of up to 480
    "n12288": (lambda: W.example41(1.5, 96, 128), 20),
    "n20000_restart7": (lambda: W.tiny(625, 32, 1.7, 2, "gbdf3"), 7),
    "n131584_chunk_limit": (lambda: W.tiny(257, 512, 1.4, 3, "trapezoidal"), 20),
}


@pytest.mark.parametrize("side", ["right", "left"])
@pytest.mark.parametrize("name", list(CASES))
def test_two_pass_mgs_solves(name, side):
    make, restart = CASES[name]
    p = make()
    assert p.m * p.s > 7168
    S = BvmSolver(p)
    S.factor("fp64")
    u, info = S.solve(p.u0, p.f, rtol=1e-10, restart=restart, side=side)
    S.set_option(N.FDE_OPT_ORTHO, N.FDE_ORTHO_CGS2)
    u2, info2 = S.solve(p.u0, p.f, rtol=1e-10, restart=restart, side=side)
    assert info["converged"] == 1 and abs(info["iters"] - info2["iters"]) <= 1
    assert _rel(u, u2) <= 1e-9
    if side == "right":
        assert info["true_relres"] <= 1e-10 and O.true_relres(p, u) <= 1.5e-10
    S.close()


def test_two_pass_mgs_with_many_basis_vectors():
    """No preconditioner, restart 64: up to 64 basis vectors, four groups a pass."""
    p = W.tiny(150, 64, 1.3, 4, "gbdf3")
    S = BvmSolver(p)
    S.factor("fp64", "none")
    u, info = S.solve(p.u0, p.f, rtol=1e-8, restart=64, maxit=4000)
    S.set_option(N.FDE_OPT_ORTHO, N.FDE_ORTHO_CGS2)
    u2, info2 = S.solve(p.u0, p.f, rtol=1e-8, restart=64, maxit=4000)
    assert info["iters"] > 64 and abs(info["iters"] - info2["iters"]) <= max(2, info["iters"] // 50)
    assert info["true_relres"] <= 1e-8
    S.close()


@pytest.mark.parametrize("restart", [20, 5])
def test_batches_mix_the_three_forms(restart):
    ps = [W.tiny(63, 16, 1.5, 1, "gbdf3"), W.tiny(200, 32, 1.7, 4, "gbdf3"), W.tiny(301, 64, 1.3, 5, "trapezoidal"),
          W.tiny(230, 32, 1.8, 6, "gbdf3")]
    batch = [BvmSolver(p) for p in ps]
    factor_batch(batch, "fp64")
    for _ in range(2):
        outs, infos = solve_batch(batch, [p.u0 for p in ps], [p.f for p in ps], restart=restart)
        for p, u, info in zip(ps, outs, infos):
            S = BvmSolver(p)
            S.factor("fp64")
            u1, i1 = S.solve(p.u0, p.f, restart=restart)
            assert np.array_equal(u, u1) and info["iters"] == i1["iters"], p.name
            S.close()
    for B in batch:
        B.close()
