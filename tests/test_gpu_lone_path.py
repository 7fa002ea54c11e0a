"""Which solves take the wires without neighbours out of the iteration, and how well they solve them: each
lone wire on its own to a hundredth of the tolerance (a tenth of that for the order of the sums), which the
residual of the whole cloud does not show.  Complex128 solves, COCG_RR and a caller's own guess keep every
wire."""
import numpy as np
import pytest

from paper_2410_03060_amd import workloads as W
from parity_util import say
from test_gpu_lone import _residual

pytestmark = pytest.mark.gpu

TOL = 1e-8


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


CASES = [(n_seg, R, method) for n_seg in (8, 20) for R, method in
         ((1, "COCG"), (4, "GMRES"), (3, "GCR"), (32, "COCG"), (33, "COCG"), (70, "COCG"))]


def _solve(B, cl, Z, P, inc, prec, method, x0=None):
    B.profile_enable(True)
    X, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat,
                      B.solve_opts(tol=TOL, prec=prec, method=getattr(B, method),
                                   restart=2000 if method.startswith("COCG") else 40), x0=x0)
    B.profile_enable(False)
    return X, info, B.profile_read()


@pytest.mark.parametrize("n_seg,R,method", CASES)
def test_complex64(B, n_seg, R, method):
    import torch
    cloud = W.random_cloud(5, 5801 if n_seg == 8 else 2200, box_lam=60.0 if n_seg == 8 else 40.0, d_c_lam=1.0, n_seg=n_seg)
    inc = W.random_incidences(np.random.default_rng(7), R)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C64)
    X, info, prof = _solve(B, cl, Z, P, inc, B.C64, method)
    deg = torch.as_tensor(np.diff(cl.pattern()[0]), device="cuda")
    n_lone, nb = int((deg == 1).sum()), cl.nb
    flops = 8 * nb * nb * n_lone * (R + 3 * nb if R > 32 else 4 * R)
    assert prof["lone_solve"]["launches"] == 1 and prof["lone_solve"]["flops"] == flops
    r2, u2 = _residual(B, cl, Z, X, inc)
    worst = (r2[deg == 1] / u2[deg == 1]).sqrt().max().item()
    say(f"[lone path] nb={nb} R={R} {method}: {n_lone} of {cl.n}, worst lone wire {worst:.1e}, all {info['max_rel_residual']:.1e}")
    assert worst <= 1.1 * 0.01 * TOL
    assert (r2.sum(0) / u2.sum(0)).sqrt().max().item() <= 1.1 * TOL
    if R <= 4:
        _, _, prof = _solve(B, cl, Z, P, inc, B.C64, method, x0=torch.zeros_like(X))
        assert "lone_solve" not in prof


@pytest.mark.parametrize("R,method", [(1, "GMRES"), (2, "COCG"), (40, "COCG")])
def test_complex128_keeps_every_wire(B, R, method):
    cloud = W.random_cloud(5, 5801, box_lam=60.0, d_c_lam=1.0)
    inc = W.random_incidences(np.random.default_rng(7), R)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C128)
    X, info, prof = _solve(B, cl, Z, P, inc, B.C128, method)
    assert "lone_solve" not in prof
    r2, u2 = _residual(B, cl, Z, X, inc)
    assert (r2.sum(0) / u2.sum(0)).sqrt().max().item() <= 1.1 * TOL
