"""Solves that take the wires without neighbours out of the iteration: against
the same solve through the general path (an explicit zero guess keeps every
wire in it), and against the stored matrix.

Bounds, from the residual targets: both solutions leave ||u - Z x|| <= tol ||u||
(checked here in FP64 from the stored blocks, with a tenth for the order of the
sums), so they differ by at most 2 tol kappa(Z) of their size; the clouds'
coupled groups are small, kappa <= 1e4.
"""
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


def _sparse(seed, n, box, d_c=1.0, n_seg=8):
    return W.random_cloud(seed, n, box_lam=box, d_c_lam=d_c, n_seg=n_seg)


def _residual(B, cl, Z, X, inc):
    """||u - Z x|| / ||u|| of every (cloud, RHS) from the stored blocks, complex128."""
    import torch
    row_ptr, col, perm, _ = cl.pattern()
    row = torch.as_tensor(np.repeat(np.arange(cl.n), np.diff(row_ptr)), device="cuda")
    col = torch.as_tensor(col.astype(np.int64), device="cuda")
    perm = torch.as_tensor(perm.astype(np.int64), device="cuda")
    R = X.shape[1]
    x = X.reshape(cl.n, cl.nb, R)[perm]
    r = B.excitation(cl, inc.k_hat, inc.e_hat).reshape(cl.n, cl.nb, R)[perm]
    u2 = (r.abs() ** 2).sum(1)
    zx = torch.zeros_like(r)
    for q in range(cl.nb):
        zx.index_add_(0, row, Z[:, :, q, None].to(torch.complex128) * x[col][:, None, q, :])
    return ((r - zx).abs() ** 2).sum(1), u2


def _check(B, cloud, R, prec, method, tol, **kw):
    inc = W.random_incidences(np.random.default_rng(7), R)
    cl = B.build_cloud(cloud)
    assert cl.n * cl.nb >= 40000 and 2 * cl.n_pairs <= 0.75 * cl.n   # the sizes that take the path
    Z, P = B.fill_Z(cl, prec)
    o = dict(tol=tol, prec=prec, method=getattr(B, method), restart=2000 if method.startswith("COCG") else 40, **kw)
    X, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(**o))
    import torch
    Xg, ig = B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(**o), x0=torch.zeros_like(X))
    say(f"[lone] N={cl.n} nb={cl.nb} pairs={cl.n_pairs} R={R} {method} {prec}: residual "
        f"{info['max_rel_residual']:.2e}, steps {info['iterations']} (general {ig['iterations']})")
    r2, u2 = _residual(B, cl, Z, X, inc)
    off = torch.zeros(cl.n, dtype=torch.int64)
    for k in range(cloud.n_clouds):
        off[cloud.cloud_off[k]:cloud.cloud_off[k + 1]] = k
    off = off.cuda()   # the internal order keeps the clouds one after the other
    rs, us = (torch.zeros((cloud.n_clouds, R), dtype=torch.float64, device="cuda").index_add_(0, off, v) for v in (r2, u2))
    rel = torch.where(us > 0, torch.sqrt(rs / us.clamp(min=1e-300)), us).cpu().numpy()
    assert rel.max() <= 1.1 * tol and info["max_rel_residual"] <= tol
    assert np.abs(rel - info["rel_res"]).max() <= 0.1 * tol
    d = (torch.linalg.norm(X - Xg) / torch.linalg.norm(Xg)).item()
    assert d <= 2 * tol * 1e4, d
    B.destroy(cl)


@pytest.mark.parametrize("R,prec,method", [(1, "C128", "GMRES"), (3, "C64", "GCR"), (5, "C64", "COCG"),
                                           (64, "C64", "COCG"), (70, "C64", "COCG"), (20, "C64", "COCG_RR"),
                                           (2, "C128", "COCG")])
def test_eight_segments(B, R, prec, method):
    cloud = _sparse(5, 5801, 60.0)
    _check(B, cloud, R, getattr(B, prec), method, 1e-8 if prec == "C64" else 1e-11)


@pytest.mark.parametrize("R,method", [(1, "COCG"), (33, "COCG"), (2, "GMRES")])
def test_twenty_segments(B, R, method):
    _check(B, _sparse(6, 2200, 40.0, n_seg=20), R, B.C64, method, 1e-8)


@pytest.mark.parametrize("use_x0", [0, 2])
def test_several_clouds(B, use_x0):
    """A cloud without a pair, a coupled one, an empty one, a single wire and a sparse one."""
    far = W.single_cloud(np.arange(40)[:, None] * np.array([[1.0, 0.0, 0.0]]), np.tile([0.0, 0.0, 1.0], (40, 1)),
                         np.full(40, 0.05), d_c=0.1)
    one = W.single_cloud(np.zeros((1, 3)), np.array([[0.0, 1.0, 0.0]]), np.array([0.05]), d_c=0.1)
    parts = [far, _sparse(8, 300, 9.0), one, _sparse(9, 6000, 70.0)]
    cloud = W.concat_clouds(parts)
    off = cloud.cloud_off
    cloud.cloud_off = np.array([off[0], off[1], off[2], off[2], off[3], off[4]], dtype=np.int64)   # an empty cloud
    _check(B, cloud, 9, B.C64, "COCG", 1e-8, use_x0=use_x0)


def test_no_pairs_at_all(B):
    n = 5800
    g = np.stack(np.meshgrid(np.arange(18), np.arange(18), np.arange(18), indexing="ij"), -1).reshape(-1, 3)[:n] * 0.3
    rng = np.random.default_rng(3)
    t = rng.standard_normal((n, 3))
    cloud = W.single_cloud(g, t / np.linalg.norm(t, axis=1, keepdims=True), rng.uniform(0.04, 0.06, n), d_c=0.1)
    inc = W.azimuth_incidences(3)
    cl = B.build_cloud(cloud)
    assert cl.n_pairs == 0
    Z, P = B.fill_Z(cl, B.C64)
    X, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(tol=1e-9))
    r2, u2 = _residual(B, cl, Z, X, inc)
    rel = (r2.sum(0) / u2.sum(0)).sqrt().cpu().numpy()
    assert rel.max() <= 1e-9 and np.abs(rel - info["rel_res"][0]).max() <= 1e-10


def test_a_preconditioner_that_is_not_the_inverse(B):
    """The block inverses are the caller's buffer: where they do not solve the lone wires, the
    call goes through the general path and still reaches its residual."""
    cloud = _sparse(5, 5801, 60.0)
    inc = W.azimuth_incidences(2)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C64)
    X, info = B.solve(cl, Z, P * 0.25, inc.k_hat, inc.e_hat,
                      B.solve_opts(tol=1e-7, method=B.COCG, restart=2000, inner_tol=1e-3))
    assert info["max_rel_residual"] <= 1e-7
    r2, u2 = _residual(B, cl, Z, X, inc)
    assert (r2.sum(0) / u2.sum(0)).sqrt().max().item() <= 1.1e-7
    # a block of a lone wire that is not finite is reported, never counted as solved
    row_ptr, _, _, _ = cl.pattern()
    i = int(np.nonzero(np.diff(row_ptr) == 1)[0][0])
    Z[int(row_ptr[i]), 0, 0] = complex(float("nan"), 0.0)
    with pytest.raises(B.ChaffError) as err:
        B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(tol=1e-6, method=B.COCG, restart=50, max_cycles=3))
    assert err.value.status == B.ENOCONV


def test_a_preconditioner_that_is_not_the_inverse_many_columns(B):
    """The same where the inverses are refined once per wire."""
    cloud = _sparse(5, 5801, 60.0)
    inc = W.azimuth_incidences(40)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C64)
    X, info = B.solve(cl, Z, P * 0.25, inc.k_hat, inc.e_hat,
                      B.solve_opts(tol=1e-7, method=B.COCG, restart=2000, inner_tol=1e-3))
    assert info["max_rel_residual"] <= 1e-7
    r2, u2 = _residual(B, cl, Z, X, inc)
    assert (r2.sum(0) / u2.sum(0)).sqrt().max().item() <= 1.1e-7
    row_ptr, _, _, _ = cl.pattern()
    i = int(np.nonzero(np.diff(row_ptr) == 1)[0][0])
    Z[int(row_ptr[i]), 0, 0] = complex(float("nan"), 0.0)
    with pytest.raises(B.ChaffError) as err:
        B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(tol=1e-6, method=B.COCG, restart=50, max_cycles=3))
    assert err.value.status == B.ENOCONV
