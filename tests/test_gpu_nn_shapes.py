"""Gradients of the warm-start network at layer shapes around its product kernel's choices: 64- and
16-wide tiles, vector and element-wise loads, ragged tiles and K steps, split products, the
convolutions' zero-padded input rows read in place through a row index, and bias sums over more
than one 256-row stage with a remainder.  Reference and tolerance as for the fixed small network:
the FP64 NumPy network with every product operand rounded to bf16, each tensor within 1e-2."""
import numpy as np
import pytest

import workloads as W
from oracle import nn as R
from paper_1305_6653_amd import warmstart as WS

pytestmark = pytest.mark.gpu


def _bf16(x):
    u = np.asarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) >> 16 << 16
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


SHAPES = {
    "ragged_vector_loads": (dict(m=37, s=12, conv_ch=(20, 12, 8), fc=(40, 24), nx=5, nt=4), 5),
    "odd_channels": (dict(m=21, s=9, conv_ch=(7, 5, 3), fc=(11, 9), nx=3, nt=3), 3),
    "wide_tiles": (dict(m=15, s=8, conv_ch=(72, 8, 6), fc=(20, 12), nx=4, nt=3), 64),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_gradients_at_tile_and_stage_edges(name):
    import torch
    shape, B = SHAPES[name]
    dev = torch.device("cuda:0")
    net = WS.WarmStartNet(max_batch=B, seed=2, **shape)
    cfg = R.NetConfig(**shape)
    rng = np.random.default_rng(8)
    theta = (rng.standard_normal(net.num_params) * 0.3).astype(np.float32)
    net.set_params(theta)
    rows = B + 2
    ps = [W.random_instance(700 + i, m=shape["m"], s=8, zero_u0=True) for i in range(rows)]
    for p in ps:  # the network takes any s; the instances' f is resampled in time
        p.f = np.ascontiguousarray(p.f[np.arange(shape["s"] + 1) % 9])
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to(dev)
    X = torch.zeros((rows, 256, net.cin), dtype=torch.float32, device=dev)
    rms = torch.zeros(rows, dtype=torch.float32, device=dev)
    for b0 in range(0, rows, B):
        q = ps[b0:b0 + B]
        net.features([d(p.f) for p in q], [d(p.d_plus) for p in q], [d(p.d_minus) for p in q],
                     [p.alpha for p in q], X, rms, row0=b0)
    T = rng.standard_normal((rows, shape["s"] * shape["m"]))
    idx = rng.permutation(rows)[:B].astype(np.int32)
    loss = net.loss_grad(X, d(T), rms, idx, B)
    g = net.get(1)
    feats = [R.features(cfg, ps[i].f, ps[i].d_plus, ps[i].d_minus, ps[i].alpha) for i in idx]
    loss_r, g_r = R.loss_and_grad(cfg, theta.astype(np.float64), [x for x, _ in feats], [T[i] for i in idx],
                                  [r for _, r in feats], q=_bf16)
    assert abs(loss - loss_r) <= 1e-2 * loss_r, (loss, loss_r)
    for li, ((gW, gb), (rW, rb)) in enumerate(zip(R.unpack(cfg, g.astype(np.float64)), R.unpack(cfg, g_r))):
        for what, a, b in (("W", gW, rW), ("b", gb, rb)):
            err = np.linalg.norm(a - b) / np.linalg.norm(b)
            assert err <= 1e-2, (li, what, err)
    net.close()
