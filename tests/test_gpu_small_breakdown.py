"""An excitation that is not finite in a small solve: its currents are not finite either (the lockstep
solver's become so as soon as another system takes a step), its residual is +inf, and the other systems of
the call have the currents that they have without it."""
import math

import numpy as np
import pytest

from paper_2410_03060_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("method", ["GMRES", "COCG"])
@pytest.mark.parametrize("prec", ["C64", "C128"])
@pytest.mark.parametrize("x0", [0, 2])
@pytest.mark.parametrize("value", [math.nan, math.inf])
def test_one_wave_is_not_finite(B, method, prec, x0, value):
    cloud = W.random_cloud(2, 120, box_lam=9.0, d_c_lam=1.5)   # with lone wires
    inc = W.random_incidences(np.random.default_rng(5), 3)
    cl = B.build_cloud(cloud)
    p = getattr(B, prec)
    Z, P = B.fill_Z(cl, p)
    o = dict(tol=1e-6, method=getattr(B, method), prec=p, use_x0=x0, restart=200 if method == "COCG" else 30)
    good, _ = B.solve(cl, Z, P, inc.k_hat, inc.e_hat, B.solve_opts(**o))
    eh = inc.e_hat.copy()
    eh[1, 0] = value
    B.profile_enable(True)
    X, info = B.solve(cl, Z, P, inc.k_hat, eh, B.solve_opts(**o), raise_on_noconv=False)
    B.profile_enable(False)
    assert "solve_small" in B.profile_read()
    assert info["status"] == B.ENOCONV and math.isinf(info["rel_res"][0, 1])
    X, good = X.cpu().numpy(), good.cpu().numpy()
    assert not np.isfinite(X[:, 1]).any()
    assert np.array_equal(X[:, [0, 2]], good[:, [0, 2]])
