"""Which side of the one-launch rule a call falls on: the Krylov basis and the rows of a system count
beside its blocks, and of several clouds the largest one counts.  Either way the residual of the stored
blocks is at most the tolerance (a tenth for the order of the sums)."""
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


def _box(n, seed=2):
    return W.random_cloud(seed, n, box_lam=10.0 * (n / 64.0) ** (1.0 / 3.0), d_c_lam=1.5)


def _sparse(n):
    return W.random_cloud(3, n, box_lam=25.0 * (n / 1000.0) ** (1.0 / 3.0), d_c_lam=1.0)


CALLS = [  # cloud, precision, method, restart, one launch?
    ("sparse_1000", lambda: _sparse(1000), "C128", "GMRES", 200, False),
    ("sparse_1000", lambda: _sparse(1000), "C128", "GMRES", 30, True),
    ("box_300", lambda: _box(300), "C128", "GMRES", 200, True),
    ("box_900", lambda: _box(900), "C128", "COCG", 2000, False),
    ("box_600", lambda: _box(600), "C128", "COCG", 2000, True),
    ("box_900", lambda: _box(900), "C64", "COCG", 2000, True),
    ("twelve_100", lambda: W.concat_clouds([_sparse(100) for _ in range(12)]), "C128", "COCG", 2000, True),
]


@pytest.mark.parametrize("name,make,prec,method,restart,small", CALLS,
                         ids=[f"{c[0]}-{c[2]}-{c[3]}{c[4]}" for c in CALLS])
def test_route(B, name, make, prec, method, restart, small):
    cloud = make()
    inc = W.random_incidences(np.random.default_rng(1), 2)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, getattr(B, prec))
    tol = 1e-6 if prec == "C64" else 1e-10
    B.profile_enable(True)
    X, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat,
                      B.solve_opts(tol=tol, prec=getattr(B, prec), method=getattr(B, method), restart=restart))
    B.profile_enable(False)
    say(f"[route] {name} {prec} {method}({restart}): {cl.nnzb} blocks, {info['iterations']} steps")
    assert ("solve_small" in B.profile_read()) == small
    r2, u2 = _residual(B, cl, Z, X, inc)
    off = cloud.cloud_off
    for k in range(cloud.n_clouds):   # the internal order keeps the clouds one after the other
        rel = (r2[off[k]:off[k + 1]].sum(0) / u2[off[k]:off[k + 1]].sum(0)).sqrt()
        assert rel.max().item() <= 1.1 * tol and info["rel_res"][k].max() <= tol
