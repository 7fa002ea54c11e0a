"""Solves of two host threads at once, each on a stream of its own: their step counts come through slots
of their own, so every solve has the bits that it has alone."""
import threading

import numpy as np
import pytest

from paper_2410_03060_amd import workloads as W
from parity_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


def test_two_threads(B):
    import torch
    jobs = []
    for seed, n, R, precond in ((1, 1500, 5, False), (2, 1300, 9, True)):
        cl = B.build_cloud(W.random_cloud(seed, n, box_lam=9.0, d_c_lam=1.5))
        Z, P = B.fill_Z(cl, B.C64)
        inc = W.random_incidences(np.random.default_rng(seed), R)
        kh, eh = (torch.as_tensor(v, device="cuda") for v in (inc.k_hat, inc.e_hat))
        M = B.nbhd_precond(cl, Z, 4) if precond else P
        o = dict(tol=1e-6, inner_tol=1e-5, method=B.COCG, restart=2000,
                 precond=B.PRECOND_NBHD if precond else B.PRECOND_BLOCK)
        jobs.append(lambda cl=cl, Z=Z, M=M, kh=kh, eh=eh, o=o: B.solve(cl, Z, M, kh, eh, B.solve_opts(**o)))
    alone = [job() for job in jobs]
    torch.cuda.synchronize()
    wrong, steps = [], [0, 0]

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(12):
                    X, info = jobs[k]()
                    steps[k] += info["iterations"]
                    if info["iterations"] != alone[k][1]["iterations"] or not torch.equal(X, alone[k][0]):
                        wrong.append((k, info))
                torch.cuda.current_stream().synchronize()
        except Exception as e:   # a thread's own failure is the test's
            wrong.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    say(f"[threads] {steps} steps in 12 solves each")
    assert not wrong, wrong[0]
