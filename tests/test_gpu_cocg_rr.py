"""COCG with residual replacement keeps every wire in its recurrence: on the coupled wires alone its FP32
recurrences broke down on clouds that it solves with all of them."""
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


def test_sparse_clouds_of_five_columns(B):
    steps = []
    for seed in range(16):
        cl = B.build_cloud(W.random_cloud(seed, 5801, box_lam=60.0, d_c_lam=1.0))
        Z, P = B.fill_Z(cl, B.C64)
        inc = W.random_incidences(np.random.default_rng(7 + seed), 5)
        B.profile_enable(True)
        _, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat,
                          B.solve_opts(tol=1e-6, method=B.COCG_RR, restart=2000, max_cycles=20), raise_on_noconv=False)
        B.profile_enable(False)
        steps.append(info["iterations"])
        assert info["status"] == B.OK, (seed, info)
        assert "lone_solve" not in B.profile_read()
        B.destroy(cl)
    say(f"[cocg_rr] steps {steps}")
