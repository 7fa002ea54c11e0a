"""Gradients of the training pass at the edges of its row tiles: one row, a tile
and one more, and the batches at which a workgroup takes 32 and 64 rows; the
bounds are those of the BF16-emulating comparison in test_gpu_mlp.py."""
import numpy as np
import pytest

from oracle import mlp as omlp
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


@pytest.mark.parametrize("rows,gather", [(1, True), (16, False), (17, True), (15873, True), (32257, False)])
def test_gradient_at_tile_edges(B, rows, gather):
    import torch
    rng = np.random.default_rng(rows)
    pool = rows + 100
    X = omlp.bf16(rng.standard_normal((pool, omlp.N_FEAT)))
    T = rng.standard_normal((pool, omlp.N_OUT)).astype(np.float32).astype(np.float64)
    idx = rng.permutation(pool)[:rows] if gather else np.arange(rows)
    th = W.mlp_init(7).astype(np.float32).astype(np.float64)
    g, loss = B.mlp_grad(torch.from_numpy(th.astype(np.float32)).cuda(),
                         torch.from_numpy(omlp.bf16_bits(X).view(np.int16)).cuda(),
                         torch.from_numpy(T.astype(np.float32)).cuda(),
                         torch.from_numpy(idx.astype(np.int64)).cuda() if gather else None, n_rows=rows)
    g = g.cpu().numpy().astype(np.float64)
    le, ge = omlp.loss_and_grad(th, X[idx], T[idx], emulate_bf16=True)
    assert abs(float(loss.item()) - le) <= 1e-3 * le
    lay, _ = omlp.param_layout()
    for w, b, i, o in lay:
        for sl in (slice(w, w + i * o), slice(b, b + o)):
            a, e = g[sl], ge[sl]
            cos, rel = a @ e / (np.linalg.norm(a) * np.linalg.norm(e)), np.linalg.norm(a - e) / np.linalg.norm(e)
            assert cos >= 0.9999 and rel <= 1e-2, (sl, cos, rel)
    say(f"[mlp rows] {rows} gather={gather}: loss {le:.3e}")
