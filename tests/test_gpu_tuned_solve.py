"""The recorded product variant inside solves that iterate on the coupled wires alone: the entry of the
whole cloud counts, as if the options named it, and an entry that happens to carry the sizes of the
coupled wires does not.  The variants add in different orders, so equal bits tell which one ran."""
import json

import numpy as np
import pytest

from paper_2410_03060_amd import workloads as W
from parity_util import say

pytestmark = pytest.mark.gpu

S = 3


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


def _record(B, path, n, nnzb, best):
    path.write_text(json.dumps([dict(nb=7, n=int(n), nnzb=int(nnzb), s=S, prec=0, best=best, ms=[1.0] * 8)]))
    assert B.tune_load(str(path)) == 1


@pytest.mark.parametrize("method", ["GMRES", "GCR"])
def test_the_whole_clouds_entry_counts(B, tmp_path, method):
    cloud = W.random_cloud(5 if method == "GMRES" else 6, 5801, box_lam=60.0, d_c_lam=1.0)
    inc = W.random_incidences(np.random.default_rng(7), S)
    cl = B.build_cloud(cloud)
    Z, P = B.fill_Z(cl, B.C64)

    def solve(variant):
        B.profile_enable(True)
        X, _ = B.solve(cl, Z, P, inc.k_hat, inc.e_hat,
                       B.solve_opts(tol=1e-8, method=getattr(B, method), spmm_variant=variant))
        B.profile_enable(False)
        assert "lone_solve" in B.profile_read()
        return X.cpu().numpy()

    named = {v: solve(v) for v in (0, 6, 7)}
    assert not np.array_equal(named[0], named[7])
    rule = solve(-1)
    assert np.array_equal(rule, named[6])   # three columns on short rows
    deg = np.diff(cl.pattern()[0])
    coupled = int((deg > 1).sum())
    say(f"[tuned] {method}: {coupled} of {cl.n} wires coupled")
    _record(B, tmp_path / "a.json", coupled, cl.nnzb - (cl.n - coupled), 7)
    assert np.array_equal(solve(-1), rule)
    for v in (7, 0):
        _record(B, tmp_path / "b.json", cl.n, cl.nnzb, v)
        assert np.array_equal(solve(-1), named[v]), v
