"""What users of this library run, as measurable cases.

``listed()`` gives the named cases, ``draw(rng)`` one more of the same ranges.  A case is a dict
of plain values; ``prepare(case, seed)`` builds what a program holds before the call (a set-up
handle, device inputs, for some kinds a factorization or a network), ``run(state)`` is one pass
through the public entry points, ``work(case)`` what that pass cannot do without, and
``exact(case, seed)`` its result in FP64 by plain NumPy.

Kinds:
  solve    factor + solve of one system: new coefficients, one right-hand side
  resolve  solve only: the factorization is kept, the right-hand side is new
  precond  one application of the preconditioner to a vector (the step of a caller's own
           Krylov method)
  batch    factor + solve of several uneven systems at once
  train    four epochs of warm-start training over 128 instances, and the parameters
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

from paper_1305_6653_amd import BvmSolver, factor_batch, solve_batch

#: the widest block factors of a listed case, s/2+1 blocks of order 4096
_MOST_FACTOR = 129 * 4096 ** 2


def listed():
    solve = {"kind": "solve", "rtol": 1e-10, "side": "right", "precond": "strang", "data": "smooth"}
    return [
        # the 63 x 64 manufactured-solution size: the smallest ordinary call, all launch latency
        {**solve, "name": "solve_63x64_trap", "m": 63, "s": 64, "alpha": 1.5, "bvm": "trapezoidal", "prec": "fp64"},
        # a row of the iteration tables of Example 4.1: fifth-order GAM, left preconditioning
        {**solve, "name": "table_96x64_gam5", "m": 96, "s": 64, "alpha": 1.5, "bvm": "gam5", "prec": "fp64",
         "rtol": 1e-8, "side": "left", "data": "pulse"},
        # the same table's circulant preconditioner (no block factors, more iterations)
        {**solve, "name": "table_96x128_gam5_bccb", "m": 96, "s": 128, "alpha": 1.2, "bvm": "gam5", "prec": "fp64",
         "rtol": 1e-8, "side": "left", "precond": "bccb", "data": "pulse"},
        # the warm-start grid: an ordinary desktop-sized problem
        {**solve, "name": "solve_255x128", "m": 255, "s": 128, "alpha": 1.4, "bvm": "gbdf3", "prec": "fp64",
         "data": "tanh"},
        # an odd size between the tuned ones, short time axis
        {**solve, "name": "solve_701x64", "m": 701, "s": 64, "alpha": 1.7, "bvm": "gbdf3", "prec": "fp64"},
        # the 1023 x 512 benchmark workload
        {**solve, "name": "solve_1023x512", "m": 1023, "s": 512, "alpha": 1.8, "bvm": "gbdf3", "prec": "fp64"},
        # the 4095 x 256 benchmark workload in both precisions: the largest calls
        {**solve, "name": "solve_4095x256", "m": 4095, "s": 256, "alpha": 1.3, "bvm": "gbdf3", "prec": "fp64"},
        {**solve, "name": "solve_4095x256_mixed", "m": 4095, "s": 256, "alpha": 1.3, "bvm": "gbdf3", "prec": "mixed"},
        # one application of the preconditioner, the step of a caller's own Krylov method
        {**solve, "kind": "precond", "name": "precond_1000x128", "m": 1000, "s": 128, "alpha": 1.5, "bvm": "gbdf3",
         "prec": "fp64"},
        # many right-hand sides against one factorization, a ragged large grid
        {**solve, "kind": "resolve", "name": "resolve_1900x128", "m": 1900, "s": 128, "alpha": 1.6, "bvm": "gbdf3",
         "prec": "fp64", "data": "tanh"},
        # an uneven batch in the mixed form (sizes of the 64-instance batch workload)
        {"kind": "batch", "name": "batch8_mixed", "sizes": "127x64,255x256,511x128,1023x64,2047x64,127x512,255x128,511x512",
         "prec": "mixed", "rtol": 1e-10, "data": "tanh", "bvm": "gbdf3"},
        # warm-start training on the 255 x 128 grid
        {"kind": "train", "name": "train_255x128", "m": 255, "s": 128, "batch": 64},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "solve", "resolve", "precond", "batch"])
    prec = rng.choice(["fp64", "fp64", "mixed"])
    alpha = round(rng.uniform(1.1, 1.9), 3)
    if kind == "batch":
        sizes = ["%dx%d" % (_log_int(rng, 64, 1600), 2 ** rng.randint(4, 8)) for _ in range(rng.randint(2, 8))]
        return {"kind": "batch", "sizes": ",".join(sizes), "prec": prec, "rtol": 1e-10, "data": "tanh", "bvm": "gbdf3"}
    bvm = rng.choice(["trapezoidal", "gbdf3", "gbdf3", "gam5"])
    data = rng.choice(["smooth", "tanh", "pulse"])
    left = kind == "solve" and rng.random() < 0.2
    if kind == "precond" or left or data == "pulse":
        # a single application in the mixed form is an FP32 result that only its own flexible
        # GMRES uses; the tables of Example 4.1 (the pulse, left preconditioning) are FP64
        prec = "fp64"
    while True:
        m, s = _log_int(rng, 24, 4095), 2 ** rng.randint(4, 9)
        if (s // 2 + 1) * m * m <= _MOST_FACTOR:
            break
    return {"kind": kind, "m": m, "s": s, "alpha": alpha, "bvm": bvm, "prec": prec, "rtol": 1e-8 if left else 1e-10,
            "side": "left" if left else "right", "precond": "strang", "data": data}


# ---- inputs -----------------------------------------------------------------------------
def _sines(x, count):
    return np.sin(np.outer(np.arange(1, count + 1), np.pi * x / 2.0))


def _problem(m, s, alpha, bvm, data, rng):
    """One instance of u_t = d+ D+^a u + d- D-^a u + f on (0, 2) x (0, 1], time-major f."""
    x = 2.0 / (m + 1) * np.arange(1, m + 1)
    t = np.arange(s + 1) / s
    if data == "pulse":  # Example 4.1: constant coefficients, a Gaussian pulse, no source
        at = 1.2 + 0.1 * rng.uniform(-1.0, 1.0)
        return types.SimpleNamespace(
            alpha=alpha, m=m, s=s, bvm=bvm, d_plus=np.full(m, 0.6), d_minus=np.full(m, 0.5),
            f=np.zeros((s + 1, m)), u0=np.exp(-((x - at) ** 2) / (2.0 * 0.08 ** 2)))
    if data == "smooth":
        base = 1.0 + 0.5 * np.sin(np.pi * x / 2.0)
        d_plus, d_minus = base + rng.uniform(-0.1, 0.1, m), base + rng.uniform(-0.1, 0.1, m)
    else:
        e = rng.standard_normal((2, 6)) / np.arange(1, 7)
        d_plus, d_minus = 1.0 + 0.5 * np.tanh(e @ _sines(x, 6))
    p, q = np.arange(1, 9)[:, None], np.arange(5)[None, :]
    a = rng.standard_normal((8, 5)) / (p ** 2 * (1.0 + q ** 2))
    f = np.cos(np.outer(t, np.pi * np.arange(5))) @ (a.T @ _sines(x, 8))
    u0 = (rng.standard_normal(8) / np.arange(1, 9) ** 2) @ _sines(x, 8)
    return types.SimpleNamespace(alpha=alpha, m=m, s=s, bvm=bvm, d_plus=d_plus, d_minus=d_minus, f=f, u0=u0)


def _instances(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] == "batch":
        out = []
        for size in case["sizes"].split(","):
            m, s = map(int, size.split("x"))
            out.append(_problem(m, s, float(rng.uniform(1.1, 1.9)), case["bvm"], case["data"], rng))
        return out
    return [_problem(case["m"], case["s"], case["alpha"], case["bvm"], case["data"], rng)]


def _vector(case, seed):
    return np.random.default_rng((seed, 1)).standard_normal((case["s"], case["m"]))


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def prepare(case, seed):
    if case["kind"] == "train":
        return _prepare_training(case, seed)
    ps = _instances(case, seed)
    st = {"case": case, "solvers": [BvmSolver(p) for p in ps]}
    st["u0"] = [_dev(p.u0) for p in ps]
    st["f"] = [_dev(p.f) for p in ps]
    st["out"] = [torch.empty((p.s, p.m), dtype=torch.float64, device="cuda") for p in ps]
    if case["kind"] in ("resolve", "precond"):
        st["solvers"][0].factor(case["prec"], case["precond"])
    if case["kind"] == "precond":
        st["v"] = _dev(_vector(case, seed))
    torch.cuda.synchronize()
    return st


def _prepare_training(case, seed):
    from paper_1305_6653_amd.warmstart import WarmStartNet, build_dataset

    def make(i):
        rng = np.random.default_rng((seed, i))
        p = _problem(case["m"], case["s"], float(rng.uniform(1.1, 1.9)), "gbdf3", "tanh", rng)
        p.u0 = np.zeros(p.m)
        return p

    net = WarmStartNet(case["m"], case["s"], max_batch=case["batch"], seed=seed % 1000)
    data = build_dataset(list(range(2 * case["batch"])), net, make, batch=case["batch"])
    return {"case": case, "net": net, "data": data, "seed": seed}


def run(st):
    case = st["case"]
    if case["kind"] == "train":
        from paper_1305_6653_amd.warmstart import train
        losses = train(st["net"], st["data"], epochs=4, batch=case["batch"], seed=st["seed"])
        return {"loss": np.array(losses, dtype=np.float32), "params": st["net"].get(0)}
    S = st["solvers"]
    if case["kind"] == "batch":
        factor_batch(S, case["prec"])
        return solve_batch(S, st["u0"], st["f"], outs=st["out"], rtol=case["rtol"])[0]
    if case["kind"] == "precond":
        return S[0].precond(st["v"], out=st["out"][0])
    if case["kind"] == "solve":
        S[0].factor(case["prec"], case["precond"])
    return S[0].solve(st["u0"][0], st["f"][0], out=st["out"][0], rtol=case["rtol"], side=case["side"])[0]


# ---- what a pass cannot do without ------------------------------------------------------
def _minimum(m, s, vectors):
    """Inputs and outputs once; a product with J at every time level by FFTs of twice the grid
    and the time transforms of one application of the preconditioner."""
    size = 2 ** math.ceil(math.log2(max(2 * m - 1, 2)))
    flops = s * 2 * 5.0 * size * math.log2(size) + 2 * m * 2.5 * s * math.log2(s)
    return {"bytes": 8.0 * vectors, "flops": flops}


def work(case):
    if case["kind"] == "train":
        # 8 steps of about 2.5 M parameters: forward and two backward products per instance
        # (the three convolutions read 128, 64 and 32 positions, the dense layers one)
        cin, ch, fc, coef = case["s"] + 4, (96, 96, 64), (768, 512), 32 * 16
        conv = 5 * (128 * cin * ch[0] + 64 * ch[0] * ch[1] + 32 * ch[1] * ch[2])
        dense = 32 * ch[2] * fc[0] + fc[0] * fc[1] + fc[1] * coef
        basis = coef * case["s"] * case["m"]
        params = 5 * (cin * ch[0] + ch[0] * ch[1] + ch[1] * ch[2]) + dense
        inst = 256 * cin * 4 + case["s"] * case["m"] * 8
        steps = 8
        return {"bytes": float(steps * (case["batch"] * inst + params * 24) + basis * 2),
                "flops": float(steps * case["batch"] * (6 * (conv + dense) + 4 * basis))}
    if case["kind"] == "batch":
        sizes = [tuple(map(int, t.split("x"))) for t in case["sizes"].split(",")]
    else:
        sizes = [(case["m"], case["s"])]
    total = {"bytes": 0.0, "flops": 0.0}
    for m, s in sizes:
        vectors = 2 * s * m if case["kind"] == "precond" else (2 * s + 4) * m
        for k, v in _minimum(m, s, vectors).items():
            total[k] += v
    return total


# ---- the same results in plain FP64 NumPy -----------------------------------------------
def _space_matrix(p):
    g = np.empty(p.m + 1)
    g[0] = 1.0
    for k in range(1, p.m + 1):
        g[k] = g[k - 1] * (1.0 - (p.alpha + 1.0) / k)
    i = np.arange(p.m)
    d = i[:, None] - i[None, :] + 1
    G = np.where(d >= 0, g[np.clip(d, 0, p.m)], 0.0)
    return (2.0 / (p.m + 1)) ** -p.alpha * (p.d_plus[:, None] * G + p.d_minus[:, None] * G.T)


def _lagrange_weights(nodes, lo, hi):
    """Integrals over [lo, hi] of the Lagrange basis polynomials of ``nodes``."""
    out = []
    for j, a in enumerate(nodes):
        c = np.array([1.0])
        for i, b in enumerate(nodes):
            if i != j:
                c = np.convolve(c, [1.0, -float(b)]) / (a - b)
        c = np.polyint(c)
        out.append(np.polyval(c, hi) - np.polyval(c, lo))
    return np.array(out)


def _derivative_row(nodes, at):
    """Weights w with sum_j w_j u(nodes_j) = u'(at), exact on cubics."""
    V = np.vander(np.array(nodes, dtype=float), 4, increasing=True).T
    rhs = np.array([0.0, 1.0, 2.0 * at, 3.0 * at ** 2])
    return np.linalg.solve(V, rhs)


def _time_matrices(bvm, s):
    """A, B [s][s+1] over u_0..u_s of rows 1..s, and the main formula's (offset, alpha, beta)."""
    A, B = np.zeros((s, s + 1)), np.zeros((s, s + 1))
    if bvm == "trapezoidal":
        main = (1, np.array([-1.0, 1.0]), np.array([0.5, 0.5]))
        for n in range(1, s + 1):
            A[n - 1, n - 1:n + 1], B[n - 1, n - 1:n + 1] = main[1], main[2]
    elif bvm == "gbdf3":
        main = (2, _derivative_row([-2, -1, 0, 1], 0), np.array([0.0, 0.0, 1.0, 0.0]))
        A[0, 0:4], B[0, 1] = _derivative_row([0, 1, 2, 3], 1), 1.0
        for n in range(2, s):
            A[n - 1, n - 2:n + 2], B[n - 1, n] = main[1], 1.0
        A[s - 1, s - 3:s + 1], B[s - 1, s] = _derivative_row([-3, -2, -1, 0], 0), 1.0
    else:
        main = (2, np.array([0.0, -1.0, 1.0, 0.0, 0.0]), _lagrange_weights([-2, -1, 0, 1, 2], -1, 0))
        for n in range(1, s + 1):
            c = min(max(n, 2), s - 2)
            A[n - 1, n - 1:n + 1] = [-1.0, 1.0]
            B[n - 1, c - 2:c + 3] = _lagrange_weights([-2, -1, 0, 1, 2], n - 1 - c, n - c)
    return A, B, main


def _exact_solve(p):
    """The all-at-once system by the eigenvectors of J and one s x s system per eigenvalue,
    then refinement with the dense J."""
    J = _space_matrix(p)
    Ah, Bh, _ = _time_matrices(p.bvm, p.s)
    tau = 1.0 / p.s
    A, B = Ah[:, 1:], Bh[:, 1:]
    b = tau * (Bh @ p.f) - np.outer(Ah[:, 0], p.u0) + tau * np.outer(Bh[:, 0], J @ p.u0)
    lam, X = np.linalg.eig(J)
    Xi = np.linalg.inv(X)
    step = max(1, int(2e7) // p.s ** 2)

    def solve(r):
        c = (r @ Xi.T).T.astype(complex)
        for i in range(0, p.m, step):
            K = A[None] - tau * lam[i:i + step, None, None] * B[None]
            c[i:i + step] = np.linalg.solve(K, c[i:i + step, :, None])[:, :, 0]
        return (X @ c).T.real

    u = np.zeros_like(b)
    for _ in range(3):
        u = u + solve(b - A @ u + tau * (B @ u) @ J.T)
    return u


def _exact_precond(p, v):
    """S^{-1} v: the time DFT and one dense solve per frequency."""
    J = _space_matrix(p)
    _, _, (nu, al, be) = _time_matrices(p.bvm, p.s)
    ca, cb = np.zeros(p.s), np.zeros(p.s)
    for i in range(len(al)):
        ca[(nu - i) % p.s] += al[i]
        cb[(nu - i) % p.s] += be[i]
    lam, mu = np.fft.fft(ca), np.fft.fft(cb)
    vh = np.fft.rfft(v, axis=0)
    eye = np.eye(p.m)
    zh = np.stack([np.linalg.solve(lam[k] * eye - (mu[k] / p.s) * J, vh[k]) for k in range(p.s // 2 + 1)])
    return np.fft.irfft(zh, n=p.s, axis=0)


def exact(case, seed):
    if case["kind"] == "train":
        return None
    ps = _instances(case, seed)
    if case["kind"] == "precond":
        if (case["s"] // 2 + 1) * case["m"] ** 3 > 1.0e11:
            return None
        return _exact_precond(ps[0], _vector(case, seed))
    out, left = [], 4.0e10  # operations that take some seconds
    for p in ps:
        cost = 60.0 * p.m ** 3 + 3.0 * p.m * p.s ** 3
        fits = cost <= left
        left -= cost if fits else 0.0
        out.append(_exact_solve(p) if fits else None)
    if case["kind"] != "batch":
        return out[0]
    return out if any(o is not None for o in out) else None
