"""The streaming row product (one wave per block row, up to 4 columns): rows of
one block, rows around its unroll (4 and 8 blocks), long rows, vectors that are
not 16-byte aligned, and the COCG solves that run on it.  Products against the
same blocks multiplied in complex128: FP32 sums of at most 7 x 300 terms, bound
2e-6 of the result's norm (complex64), 1e-14 (complex128)."""
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


CLOUDS = {"sparse": (700, 12.0, 1.0), "near_unroll": (600, 6.0, 1.0), "dense": (300, 4.0, math.inf), "one": (1, 1.0, 1.0)}


@pytest.mark.parametrize("prec", ["C64", "C128"])
@pytest.mark.parametrize("name", list(CLOUDS))
def test_product(B, name, prec):
    import torch
    n, box, d_c = CLOUDS[name]
    cl = B.build_cloud(W.random_cloud(21, n, box_lam=box, d_c_lam=d_c))
    p = getattr(B, prec)
    Z, _ = B.fill_Z(cl, p, with_pinv=False)
    row_ptr, col, _, _ = cl.pattern()
    row = torch.as_tensor(np.repeat(np.arange(cl.n), np.diff(row_ptr)), device="cuda")
    col = torch.as_tensor(col.astype(np.int64), device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    for s in (1, 2, 3, 4, 5):
        for shift in (0, 1):   # shift 1: the vectors start 8 (16) bytes into the buffer
            buf = torch.view_as_complex(torch.randn((cl.n * 7 * s + 1, 2), generator=g, device="cuda",
                                                    dtype=torch.float64)).to(Z.dtype)
            X = buf[shift:shift + cl.n * 7 * s].view(cl.n * 7, s)
            ref = torch.zeros((cl.n, 7, s), dtype=torch.complex128, device="cuda")
            x = X.to(torch.complex128).reshape(cl.n, 7, s)[col]
            for q in range(7):
                ref.index_add_(0, row, Z[:, :, q, None].to(torch.complex128) * x[:, None, q, :])
            for v in (-1, 7):
                Y = B.spmm(cl, Z, X, p, v).to(torch.complex128).reshape(ref.shape)
                e = (torch.linalg.norm(Y - ref) / torch.linalg.norm(ref)).item()
                assert e <= (2e-6 if prec == "C64" else 1e-14), (s, shift, v, e)
    say(f"[stream] {name} {prec}: rows of {cl.nnzb / cl.n:.1f} blocks")


@pytest.mark.parametrize("R", [1, 2, 3, 4, 5])
def test_cocg_on_few_columns(B, R):
    cloud = W.random_cloud(31, 700, box_lam=7.0, d_c_lam=1.5)
    inc = W.random_incidences(np.random.default_rng(32), R)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C64)
    M = B.nbhd_precond(cl, Z, 4)
    Zs, _ = mom.snfc_matrix(cloud)
    xo = osolve.sparse_solve(Zs, mom.excitation(cloud, inc.k_hat, inc.e_hat))
    for pre, buf in ((B.PRECOND_BLOCK, P), (B.PRECOND_NBHD, M)):
        X, info = B.solve(cl, Z, buf, inc.k_hat, inc.e_hat,
                          B.solve_opts(tol=1e-6, method=B.COCG, restart=500, inner_tol=1e-3, precond=pre))
        assert np.all(info["rel_res"] <= 1e-6)
        e = current_err(X.cpu().numpy(), xo).max()
        assert e <= 1e-4
    say(f"[stream] COCG R={R}: current err {e:.2e}")
