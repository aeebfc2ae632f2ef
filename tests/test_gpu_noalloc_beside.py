"""The allocation-free apply writes nothing of the handle's: another thread may run the handle's own
applies at the same time (their launches then alternate on the handle's stream), and both keep
their results to the bit."""
import ctypes as C
import threading

import numpy as np
import pytest

import workloads as W
from paper_1305_6653_amd import BvmSolver
from paper_1305_6653_amd import _native as N

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("m,s,compress", [(1100, 16, 1), (600, 64, 1), (300, 16, 0)])
def test_beside_the_handles_own_applies(m, s, compress, prec):
    import torch
    p = W.tiny(m, s, 1.4, 7, "gbdf3")
    S = BvmSolver(p)
    S.set_option(N.FDE_OPT_COMPRESS, compress)
    S.factor(prec, blocks=None if compress else "lu")
    assert S.get_option(N.FDE_OPT_COMPRESS_IN_USE) == compress
    rng = np.random.default_rng(2)
    v, w = (torch.from_numpy(rng.standard_normal((s, m))).cuda() for _ in range(2))
    ref_v, ref_w = S.precond(v), S.precond(w)
    torch.cuda.synchronize()
    wrong, rounds, out = [], 60, torch.empty_like(w)

    def own():
        for _ in range(rounds):
            S.precond(w, out=out)
            torch.cuda.synchronize()
            if not torch.equal(out, ref_w):
                wrong.append("own")

    t = threading.Thread(target=own)
    t.start()
    z = torch.empty_like(v)
    for _ in range(rounds):
        st = N.lib().fde_apply_precond_noalloc(S.handle, C.c_void_p(v.data_ptr()), C.c_void_p(z.data_ptr()))
        torch.cuda.synchronize()
        if st != N.FDE_OK or not torch.equal(z, ref_v):
            wrong.append("allocation-free %d" % st)
    t.join()
    assert not wrong, wrong[:4]
    S.close()
