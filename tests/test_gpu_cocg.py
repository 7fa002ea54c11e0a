"""COCG with the step's sums and scalar updates in one launch and the products
on the matrix cores, over the widths where their column tiles and groups of
lanes change: every solution against the stored matrix in complex128.

Bound, from the residual target: the solve stops at ||u - Z x|| <= tol ||u|| of
its own FP64 residual; a tenth is allowed for the order of the sums here.
"""
import numpy as np
import pytest

from paper_2410_03060_amd import workloads as W
from parity_util import say
from test_gpu_lone import _residual

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


def _solve(B, cloud, R, precond, tol=1e-8):
    import torch
    inc = W.random_incidences(np.random.default_rng(3), R)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C64)
    o = dict(tol=tol, prec=B.C64, method=B.COCG, restart=3000, inner_tol=1e-5)
    if precond == "nbhd":
        X, info = B.solve(cl, Z, B.nbhd_precond(cl, Z, 4, B.C64), inc.k_hat, inc.e_hat,
                          B.solve_opts(**o, precond=B.PRECOND_NBHD))
    else:   # a named product variant keeps small solves on the general path
        X, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(**o, spmm_variant=0))
    r2, u2 = _residual(B, cl, Z, X, inc)
    off = torch.zeros(cl.n, dtype=torch.int64)
    for k in range(cloud.n_clouds):
        off[cloud.cloud_off[k]:cloud.cloud_off[k + 1]] = k
    off = off.cuda()
    rs, us = (torch.zeros((cloud.n_clouds, R), dtype=torch.float64, device="cuda").index_add_(0, off, v) for v in (r2, u2))
    rel = torch.where(us > 0, torch.sqrt(rs / us.clamp(min=1e-300)), us).cpu().numpy()
    say(f"[cocg] N={cl.n} pairs={cl.n_pairs} clouds={cloud.n_clouds} R={R} {precond}: residual {rel.max():.2e}, "
        f"steps {info['iterations']}")
    assert rel.max() <= 1.1 * tol and info["max_rel_residual"] <= tol
    assert np.abs(rel - info["rel_res"]).max() <= 0.1 * tol
    B.destroy(cl)


@pytest.mark.parametrize("precond", ["block", "nbhd"])
@pytest.mark.parametrize("R", [1, 2, 3, 5, 8, 9, 17, 33, 64, 65, 130])
def test_widths(B, R, precond):
    clouds = [W.random_cloud(11 + k, n, box_lam=b, d_c_lam=1.0) for k, (n, b) in enumerate([(1, 1.0), (37, 2.5), (1100, 8.5)])]
    _solve(B, W.concat_clouds(clouds), R, precond)


@pytest.mark.parametrize("R", [6, 64])
def test_rows_of_many_blocks(B, R):   # more than 64 blocks to a row
    _solve(B, W.random_cloud(4, 400, box_lam=8.0, d_c_lam=4.0), R, "block")
