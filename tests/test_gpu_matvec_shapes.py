"""Products with J through the circulant embedding: every transform length from 16 to 8192 (one to
four radix-8 passes on either side of a radix-2, radix-4 or radix-8 middle), node counts at the ends
of each, and row counts that leave a workgroup of several rows partly filled."""
import numpy as np
import pytest

import oracle as O
import workloads as W
from paper_1305_6653_amd import BvmSolver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 8, 9, 16, 17, 33, 64, 65, 129, 300, 512, 513, 1025, 2048, 2049, 4096])
def test_toeplitz_rows(m):
    """Normwise: a length-L FFT pair and the product by the symbol err by less than 16 log2 L eps of
    max |symbol| ||x||, and |symbol| <= sum |g| = 2 alpha."""
    p = W.tiny(m, 16, 1.5, 2, "gbdf3")
    S = BvmSolver(p)
    J = O.problem_matrices(p)[0]
    h = (p.xR - p.xL) / (m + 1)
    dmax = float(np.max(np.abs(p.d_plus) + np.abs(p.d_minus)))
    L = max(16, 2 ** int(np.ceil(np.log2(2 * m))))
    for rows in (1, 3, 16):
        x = np.random.default_rng(rows).standard_normal((rows, m))
        err = np.linalg.norm(S.toeplitz(x) - x @ J.T, axis=1)
        bound = 16 * np.log2(L) * 2.0 ** -53 * 2 * p.alpha * dmax * h ** -p.alpha * np.linalg.norm(x, axis=1)
        assert np.all(err <= bound), (rows, (err / bound).max())
    S.close()
