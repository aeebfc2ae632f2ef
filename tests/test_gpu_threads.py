"""Handles of different sizes, alphas (hence ranks) and precisions, each in a thread of its own, factored
and solved at the same time: the bits of the same work done alone."""
import threading

import numpy as np
import pytest

import workloads as W
from paper_1305_6653_amd import BvmSolver

pytestmark = pytest.mark.gpu


def test_factor_and_solve_in_threads():
    jobs = [(W.tiny(1500, 8, 1.05, 1, "gbdf3"), "fp64"), (W.tiny(1500, 8, 1.9, 2, "gbdf3"), "fp64"),
            (W.tiny(700, 16, 1.4, 3, "trapezoidal"), "mixed"), (W.tiny(90, 64, 1.6, 4, "gbdf3"), "fp64")]
    handles = [BvmSolver(p) for p, _ in jobs]
    ref = []
    for S, (p, prec) in zip(handles, jobs):
        S.factor(prec)
        ref.append(S.solve(p.u0, p.f)[0])
    wrong = []

    def work(i):
        try:
            for _ in range(12):
                handles[i].factor(jobs[i][1])
                if not np.array_equal(handles[i].solve(jobs[i][0].u0, jobs[i][0].f)[0], ref[i]):
                    wrong.append((i, "bits"))
        except Exception as e:  # seen by the assertion in the main thread
            wrong.append((i, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong[:4]
    for S in handles:
        S.close()
