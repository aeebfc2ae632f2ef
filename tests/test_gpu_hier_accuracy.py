"""A single application of S^{-1} in hierarchical form is as accurate as with the dense factors of the
same precision that it stands in for: both against block solves refined in extended precision, on
the same vectors.  FP32 blocks: no further off than the dense factors (whose entries are rounded to
FP32, an error that the form does not have).  FP64: within three times the dense error, above the
rounding of the time transforms (20 eps); for variable coefficients only.  With constant ones every
row of J is rounded alike, both errors are the sum of a few equal terms of either sign, and the
quotient of two of them is anything: over 282 applications at 100 to 1860 rows 0.02 to 7.8, its
geometric mean 0.65."""
import numpy as np
import pytest
import scipy.linalg as sl

import oracle as O
import workloads as W
from paper_1305_6653_amd import BvmSolver
from paper_1305_6653_amd import _native as N

pytestmark = pytest.mark.gpu


def _refined_apply(p, vs):
    """S^{-1} v for each v of vs: LAPACK block solves, residuals in long double."""
    J, F, tau, _ = O.problem_matrices(p)
    lam, mu = O.strang_eigs(F, p.s)
    Jl = J.astype(np.longdouble)
    vh = np.stack([np.fft.rfft(v, axis=0) for v in vs], axis=2)  # [nb][m][vectors]
    out = np.empty_like(vh)
    for k in range(p.s // 2 + 1):
        c = tau * mu[k]
        lu = sl.lu_factor(lam[k] * np.eye(p.m) - c * J)
        x = sl.lu_solve(lu, vh[k]).astype(np.clongdouble)
        for _ in range(3):
            Jx = Jl @ x.real + 1j * (Jl @ x.imag)
            r = vh[k] - (np.clongdouble(lam[k]) * x - np.clongdouble(c) * Jx)
            x = x + sl.lu_solve(lu, r.astype(complex))
        out[k] = x.astype(complex)
    return [np.fft.irfft(out[:, :, i], n=p.s, axis=0) for i in range(len(vs))]


@pytest.mark.parametrize("m,s,alpha,seed", [
    (63, 64, 1.3, 5), (300, 16, 1.1, 6), (1000, 16, 1.3, 5), (1300, 8, 1.1, 5), (1300, 8, 1.3, 5), (1800, 8, 1.1, 5),
    (1800, 8, 1.3, 5), (1800, 8, 1.5, 5), (1800, 8, 1.8, 6), (2500, 4, 1.2, 7),
    # constant coefficients (seed None): every row of J is rounded alike
    (1000, 16, 1.3, None), (1800, 8, 1.1, None), (1800, 8, 1.77, None)])
def test_no_less_accurate_than_the_dense_factors(m, s, alpha, seed):
    if seed is None:
        p = W.example41(alpha, m, s)
    else:
        p = W.random_instance(seed, m=m, s=s)
        p.alpha = alpha
    vs = [np.random.default_rng(1).standard_normal((s, m)),
          np.ones((s, 1)) * np.sin(np.pi * np.arange(1, m + 1) / (m + 1))]
    refs = _refined_apply(p, vs)
    for prec, times, floor in (("mixed", 1.0, 20 * 2.0 ** -24), ("fp64", 3.0, 20 * 2.0 ** -53)):
        if prec == "fp64" and seed is None:
            continue
        err = {}
        for compress in (0, 2):
            S = BvmSolver(p)
            S.set_option(N.FDE_OPT_COMPRESS, compress)
            S.factor(prec)
            err[compress] = [np.linalg.norm(S.precond(v) - r) / np.linalg.norm(r) for v, r in zip(vs, refs)]
            S.close()
        print(prec, m, s, alpha, "dense", err[0], "hierarchical", err[2])
        for hier, dense in zip(err[2], err[0]):
            assert hier <= max(times * dense, floor), (prec, hier, dense)
