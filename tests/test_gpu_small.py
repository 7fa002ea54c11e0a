"""Solves in one launch (few, small systems) against the oracle: both methods and
precisions, the three initial guesses, several clouds with an empty and an
uncoupled one, restarts, and the calls that end without convergence.  Bounds as
for the lockstep solver: currents 1e-4 (complex64 with refinement) and 1e-10
(complex128 at 1e-12); residuals at most the tolerance."""
import math

import numpy as np
import pytest

from oracle import mom, solve as osolve
from paper_2410_03060_amd import workloads as W
from parity_util import current_err, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


def _clouds(name):
    if name == "coupled":
        return W.random_cloud(3, 50, box_lam=4.0, d_c_lam=1.5)
    if name == "sparse":
        return W.random_cloud(4, 900, box_lam=22.0, d_c_lam=1.0)
    if name == "twenty":
        return W.random_cloud(5, 60, box_lam=9.0, d_c_lam=1.5, n_seg=20)
    far = W.single_cloud(np.arange(9)[:, None] * np.array([[1.0, 0.0, 0.0]]), np.tile([0.0, 0.0, 1.0], (9, 1)),
                         np.full(9, 0.05), d_c=1.5 * W.WAVELENGTH)
    cloud = W.concat_clouds([W.random_cloud(6, 40, box_lam=3.0, d_c_lam=1.5), far,
                             W.random_cloud(7, 300, box_lam=14.0, d_c_lam=1.5)])
    off = cloud.cloud_off
    cloud.cloud_off = np.array([off[0], off[1], off[1], off[2], off[3]], dtype=np.int64)   # with an empty cloud
    return cloud


def _launched(B, prof):
    return "solve_small" in prof and "spmm" not in prof


@pytest.mark.parametrize("name", ["coupled", "sparse", "several", "twenty"])
@pytest.mark.parametrize("method", ["GMRES", "COCG"])
@pytest.mark.parametrize("prec", ["C64", "C128"])
def test_currents(B, name, method, prec):
    cloud = _clouds(name)
    inc = W.random_incidences(np.random.default_rng(1), 3)
    cl = B.build_cloud(cloud)
    p = getattr(B, prec)
    Z, P = B.fill_Z(cl, p)
    c64 = prec == "C64"
    Zs, _ = mom.snfc_matrix(cloud, n_seg=cloud.n_seg)
    xo = osolve.sparse_solve(Zs, mom.excitation(cloud, inc.k_hat, inc.e_hat, n_seg=cloud.n_seg))
    guess = None
    for x0 in (0, 2, 1):
        o = B.solve_opts(tol=1e-6 if c64 else 1e-12, prec=p, method=getattr(B, method), use_x0=x0,
                         restart=7 if method == "GMRES" else 500, inner_tol=1e-4, max_cycles=60)
        B.profile_enable(True)
        X, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat, o, x0=guess if x0 == 1 else None)
        B.profile_enable(False)
        assert _launched(B, B.profile_read())
        assert info["rel_res"].max() <= o.tol and info["iterations"] >= info["cycles"]
        e = current_err(X.cpu().numpy(), xo).max()
        assert e <= (1e-4 if c64 else 1e-10), (x0, e)
        guess = X * 1.01
    say(f"[small] {name} {method} {prec}: current err {e:.1e}, steps {info['iterations']} in {info['cycles']} cycles")


def test_larger_calls_keep_the_lockstep_solver(B):
    cloud = W.random_cloud(8, 700, box_lam=6.0, d_c_lam=1.5)   # more blocks than one CU streams
    inc = W.azimuth_incidences(1)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C64)
    B.profile_enable(True)
    B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(tol=1e-6))
    B.profile_enable(False)
    assert "solve_small" not in B.profile_read()


@pytest.mark.parametrize("method", ["GMRES", "COCG"])
def test_no_convergence_and_breakdown(B, method):
    cloud = _clouds("sparse")
    inc = W.azimuth_incidences(2)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C64)
    o = dict(tol=1e-7, method=getattr(B, method), restart=2, max_cycles=1)
    X, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(**o), raise_on_noconv=False)
    assert info["status"] == B.ENOCONV and info["cycles"] == 1 and 1e-7 < info["max_rel_residual"] < 1
    # a preconditioner that is not the inverse: the lone wires stay in the iteration
    X, info = B.solve(cl, Z, P * 0.25, inc.k_hat, inc.e_hat,
                      B.solve_opts(tol=1e-6, method=getattr(B, method), restart=60, max_cycles=60))
    assert info["max_rel_residual"] <= 1e-6
    row_ptr, _, _, _ = cl.pattern()
    for i in (int(np.nonzero(np.diff(row_ptr) == 1)[0][0]), int(np.nonzero(np.diff(row_ptr) > 1)[0][0])):
        Zn = Z.clone()
        Zn[int(row_ptr[i]), 0, 0] = complex(float("nan"), 0.0)
        _, info = B.solve(cl, Zn, P, inc.k_hat, inc.e_hat, B.solve_opts(**dict(o, max_cycles=3)), raise_on_noconv=False)
        assert info["status"] == B.ENOCONV and math.isinf(info["max_rel_residual"])
