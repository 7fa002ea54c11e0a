"""Small solves of many steps are a row of launches: the host is back after a bounded number of steps
(512 of a system, and a GMRES cycle of at most 200 begun before them), and a launch goes on where the
last one stopped, inside a COCG cycle or between two cycles.

The block inverses are the caller's buffer; diagonal ones of very different sizes make the recurrences
slow.  Bounds: a solution with ||u - Z x|| <= tol ||u|| is off by at most tol kappa(Z) of its size; the
reported residual is the one of the stored blocks to the rounding of 64-bit sums (1e-12 of ||u||).
"""
import numpy as np
import pytest

from oracle import mom, solve as osolve
from paper_2410_03060_amd import workloads as W
from parity_util import current_err, say
from test_gpu_lone import _residual

pytestmark = pytest.mark.gpu

LAUNCH_STEPS, LONGEST_GMRES_CYCLE = 512, 200


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


def _poor(P, first, seed=1):
    """Diagonal blocks with entries from 0.1 to 10 for the wires from internal index first on."""
    import torch
    nb = P.shape[-1]
    d = 10.0 ** np.random.default_rng(seed).uniform(-1.0, 1.0, (P.shape[0], nb))
    Q = P.clone()
    Q[first:] = torch.diag_embed(torch.as_tensor(d, device="cuda", dtype=Q.dtype))[first:]
    return Q


def _solve(B, cl, Z, P, inc, **o):
    B.profile_enable(True)
    X, info = B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(**o), raise_on_noconv=False)
    B.profile_enable(False)
    return X, info, B.profile_read()["solve_small"]["launches"]


def test_a_long_cycle_goes_on_in_the_next_launch(B):
    """COCG in one cycle of over 1,000 steps, beside a cloud that is done after a few."""
    a = W.random_cloud(5, 30, box_lam=5.0, d_c_lam=1.5)
    cloud = W.concat_clouds([a, W.random_cloud(3, 60, box_lam=6.0, d_c_lam=1.5)])
    inc = W.random_incidences(np.random.default_rng(1), 2)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C128)
    X, info, launches = _solve(B, cl, Z, _poor(P, a.n), inc, tol=1e-10, prec=B.C128, method=B.COCG, restart=20000,
                               inner_tol=1e-13, max_cycles=60)
    say(f"[launches] COCG: {info['iterations']} steps in {info['cycles']} cycles, {launches} launches")
    assert info["status"] == B.OK and info["rel_res"].max() <= 1e-10
    assert info["iterations"] > 2 * LAUNCH_STEPS and launches >= info["iterations"] // LAUNCH_STEPS
    Zs, _ = mom.snfc_matrix(cloud)
    xo = osolve.sparse_solve(Zs, mom.excitation(cloud, inc.k_hat, inc.e_hat))
    kappa = np.linalg.cond(Zs.toarray() if hasattr(Zs, "toarray") else np.asarray(Zs))
    assert current_err(X.cpu().numpy(), xo).max() <= 1e-10 * kappa + 1e-10


@pytest.mark.parametrize("method,restart", [("GMRES", 1), ("GMRES", 150), ("COCG", 2)])
def test_a_solve_that_does_not_converge_returns_between_its_cycles(B, method, restart):
    cloud = W.random_cloud(3, 60, box_lam=6.0, d_c_lam=1.5)
    inc = W.random_incidences(np.random.default_rng(1), 2)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C128)
    if method == "GMRES":   # (two steps of COCG need not reduce a residual: with the inverses they do)
        P = _poor(P, 0)
    X, info, launches = _solve(B, cl, Z, P, inc, tol=1e-17, prec=B.C128, method=getattr(B, method),
                               restart=restart, inner_tol=1e-17, max_cycles=900 if restart < 100 else 20)
    say(f"[launches] {method}({restart}): {info['iterations']} steps in {info['cycles']} cycles, {launches} launches")
    assert info["status"] == B.ENOCONV
    steps = info["iterations"] + info["cycles"]
    assert steps > 2 * LAUNCH_STEPS and launches >= steps // (LAUNCH_STEPS + LONGEST_GMRES_CYCLE)
    r2, u2 = _residual(B, cl, Z, X, inc)
    rel = (r2.sum(0) / u2.sum(0)).sqrt().cpu().numpy()
    assert np.abs(rel - info["rel_res"][0]).max() <= 1e-12 * max(1.0, rel.max())
