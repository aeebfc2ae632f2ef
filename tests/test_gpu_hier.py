"""The blocks of S in hierarchical form (FDE_OPT_COMPRESS): 64-row leaves joined level by level
through low-rank couplings.  The applies are compared with the oracle's S^{-1} (LAPACK block LUs
with partial pivoting) at sizes around its leaves, levels and chunks, whole solves with the
oracle's GMRES solution, batches and the allocation-free apply with single applies bit for bit,
and the dense factors that stay readable behind it with the dense route's."""
import ctypes as C
import types

import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1305_6653_amd import BvmSolver, FdeError, factor_batch, solve_batch
from paper_1305_6653_amd import _native as N

pytestmark = pytest.mark.gpu


def _solver(p, prec, compress=2):
    S = BvmSolver(p)
    S.set_option(N.FDE_OPT_COMPRESS, compress)
    S.factor(prec)
    return S


def _rel(a, b):
    return np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b))


def _one_sided(m, s):
    """d+ = 0 on one part of the grid and d- = 0 on another (allowed while their sum is positive)."""
    p = W.tiny(m, s, 1.6, 3, "gbdf3")
    p.d_plus = p.d_plus.copy()
    p.d_minus = p.d_minus.copy()
    p.d_plus[: m // 3] = 0.0
    p.d_minus[m // 2:] = 0.0
    return p


# one leaf, two with one row, ragged last leaves, missing right halves on several levels, chunk
# boundaries (4, 8 and 16 panels), more than one level above the chunks
CASES = {
    "m1": lambda: W.tiny(1, 4, 1.3, 2, "gbdf3"),
    "m64": lambda: W.tiny(64, 8, 1.7, 3, "trapezoidal"),
    "m65": lambda: W.tiny(65, 8, 1.5, 4, "gbdf3"),
    "m130": lambda: W.tiny(130, 16, 1.2, 5, "trapezoidal"),
    "m256": lambda: W.tiny(256, 16, 1.9, 6, "gbdf3"),
    "m300": lambda: W.example41(1.2, 300, 16),
    "m511": lambda: W.tiny(511, 64, 1.05, 7, "gbdf3"),
    "m701_one_sided": lambda: _one_sided(701, 16),
    "m1100": lambda: W.random_instance(9, m=1100, s=8),
}


@pytest.mark.parametrize("prec,eps", [("fp64", 2.0 ** -53), ("mixed", 2.0 ** -24)])
@pytest.mark.parametrize("name", list(CASES))
def test_hier_preconditioner_apply(name, prec, eps):
    """Forward error of S^{-1} v within 30 eps max_k cond(K_k), the dense route's bound."""
    p = CASES[name]()
    S = _solver(p, prec)
    assert S.get_option(N.FDE_OPT_COMPRESS_IN_USE) == 1
    J, F, tau, _ = O.problem_matrices(p)
    P = O.StrangPreconditioner(J, F, p.s, tau)
    kappa = max(np.linalg.cond(P.block(k, J, tau)) for k in range(p.s // 2 + 1))
    v = np.random.default_rng(4).standard_normal((p.s, p.m))
    assert _rel(S.precond(v), P.apply(v)) <= 30 * eps * max(kappa, 10.0)
    S.close()


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-9), ("mixed", 1e-8)])
@pytest.mark.parametrize("name", ["m65", "m300", "m701_one_sided"])
def test_hier_solve_vs_oracle(name, prec, tol):
    p = CASES[name]()
    S = _solver(p, prec)
    u, info = S.solve(p.u0, p.f, rtol=1e-10)
    assert info["converged"] == 1 and info["true_relres"] <= 1e-10
    ref = O.solve_gmres(p, tol=1e-12)
    assert _rel(u, ref.x) <= tol, _rel(u, ref.x)
    D = _solver(p, prec, 0)
    assert D.get_option(N.FDE_OPT_COMPRESS_IN_USE) == 0
    _, dense = D.solve(p.u0, p.f, rtol=1e-10)
    assert abs(info["iters"] - dense["iters"]) <= 1
    D.close()
    S.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_hier_batch_equals_single(prec):
    """Instances in both forms in one batch (m = 130 stays dense by default), and refactoring, give
    the single solves' bits."""
    ps = [W.tiny(1000, 64, 1.3, 1, "gbdf3"), W.tiny(130, 32, 1.6, 2, "trapezoidal"), W.tiny(300, 16, 1.8, 3, "gbdf3")]
    batch = [BvmSolver(p) for p in ps]
    for _ in range(2):
        factor_batch(batch, prec)
        outs, infos = solve_batch(batch, [p.u0 for p in ps], [p.f for p in ps])
        for p, B, u, info, form in zip(ps, batch, outs, infos, (1, 0, 1)):
            assert B.get_option(N.FDE_OPT_COMPRESS_IN_USE) == form
            S = _solver(p, prec, 1)
            u1, i1 = S.solve(p.u0, p.f)
            assert np.array_equal(u, u1) and info["iters"] == i1["iters"], p.name
            S.close()
    for B in batch:
        B.close()


def test_hier_dense_factors_on_demand():
    """fde_get_factor_block after an automatic factorization returns the dense LU's block, and the
    solves go on in hierarchical form with the same bits; so does fde_get_hessenberg for the band."""
    p = W.tiny(300, 16, 1.4, 5, "gbdf3")
    S, D = _solver(p, "fp64", 1), _solver(p, "fp64", 0)
    u1, _ = S.solve(p.u0, p.f)
    for k in (0, 3, 8):
        assert np.array_equal(S.factor_block(k), D.factor_block(k))
    u2, _ = S.solve(p.u0, p.f)
    assert S.get_option(N.FDE_OPT_COMPRESS_IN_USE) == 1 and np.array_equal(u1, u2)
    S.factor("mixed")
    assert S.factor_block(1).shape == (300, 300)
    S.set_option(N.FDE_OPT_BLOCKS, N.FDE_BLOCKS_BAND)
    S.set_option(N.FDE_OPT_COMPRESS, 2)
    S.factor("fp64")
    H, Q = S.hessenberg()
    J = O.problem_matrices(p)[0]
    assert np.abs(Q @ H @ Q.T - J).max() <= 50 * p.m * 2.0 ** -52 * np.abs(J).max()
    S.close()
    D.close()


def test_hier_coefficients_change_and_explicit_routes():
    """fde_bvm_set_coefficients rebuilds the basis for the new alpha; an explicit dense route stays
    dense; changing the option discards the factorization; bad values are refused."""
    p, p2 = W.tiny(400, 16, 1.2, 6, "gbdf3"), W.tiny(400, 16, 1.8, 7, "gbdf3")
    S = _solver(p, "fp64", 1)
    S.set_coefficients(p2.alpha, p2.d_plus, p2.d_minus)
    S.factor("fp64")
    u, _ = S.solve(p2.u0, p2.f)
    T = _solver(p2, "fp64", 1)
    assert np.array_equal(u, T.solve(p2.u0, p2.f)[0])
    S.factor("fp64", blocks="lu")
    assert S.get_option(N.FDE_OPT_COMPRESS_IN_USE) == 0
    S.set_option(N.FDE_OPT_COMPRESS, 0)
    with pytest.raises(FdeError) as e:
        S.solve(p2.u0, p2.f)
    assert e.value.status == N.FDE_EINVAL
    with pytest.raises(FdeError):
        S.set_option(N.FDE_OPT_COMPRESS, 3)
    with pytest.raises(FdeError):
        S.set_option(N.FDE_OPT_COMPRESS_IN_USE, 1)
    S.close()
    T.close()


def test_formula_without_dominance_stays_dense():
    """u_{n+1} - u_n = tau f_n (forward Euler as a BVM): Re(lambda_k conj mu_k) < 0, so the dominance
    that the hierarchical elimination rests on is not given and the dense route is kept."""
    p = W.tiny(300, 8, 1.5, 9, "gbdf3")
    F = types.SimpleNamespace(nu=1, mu=1, alpha=[-1.0, 1.0], beta=[1.0, 0.0],
                              alpha_init=[], beta_init=[], alpha_fin=[], beta_fin=[])
    S = BvmSolver(p, formula=F)
    S.factor("fp64")
    assert S.get_option(N.FDE_OPT_COMPRESS_IN_USE) == 0
    S.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_hier_noalloc_apply_equals_the_handle_apply(prec):
    import torch
    p = W.tiny(1100, 16, 1.5, 3, "gbdf3")  # above the chunks at this s: several level launches
    S = _solver(p, prec, 1)
    assert S.get_option(N.FDE_OPT_COMPRESS_IN_USE) == 1
    v = torch.from_numpy(np.random.default_rng(1).standard_normal((p.s, p.m))).cuda()
    ref = S.precond(v)
    z = torch.full_like(v, float("nan"))
    torch.cuda.synchronize()
    st = N.lib().fde_apply_precond_noalloc(S.handle, C.c_void_p(v.data_ptr()), C.c_void_p(z.data_ptr()))
    assert st == N.FDE_OK
    torch.cuda.synchronize()
    assert torch.equal(z, ref)
    S.close()
