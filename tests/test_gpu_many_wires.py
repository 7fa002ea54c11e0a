"""Clouds whose kernels take more threads than one launch counts (2^32): the neighbour search at 32 lanes
per wire, and the products at a wave per block row.  The wires stand on a lattice wider than d_c, so the
pattern is known: every wire alone but for a few pairs.  Products are compared on rows spread over the
slices with the same rows in 64 bits; the bound is that of 7 complex FP32 terms, 32 eps."""
import numpy as np
import pytest

from paper_2410_03060_amd import workloads as W
from parity_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _give_back():
    yield
    import torch
    torch.cuda.empty_cache()

LAM = W.WAVELENGTH
GB = 1 << 30


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


def _lattice(B, n, pairs):
    """n wires, d_c of 0.1 on a lattice of spacing 1 wavelength; the last `pairs` ones beside the first."""
    import torch
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 120 * GB:
        pytest.skip("needs 120 GB of device memory")
    m = n - pairs
    side = int(np.ceil(m ** (1.0 / 3.0)))
    i = torch.arange(m, device="cuda")
    c = torch.empty((n, 3), dtype=torch.float64, device="cuda")
    for d in range(3):
        c[:m, d] = (i // side ** d % side).double() * LAM
    del i
    c[m:] = c[:pairs]
    c[m:, 2] += 0.05 * LAM
    t = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    t[:, 0] = 1.0
    L = torch.full((n,), 0.5 * LAM, dtype=torch.float64, device="cuda")
    return B.DeviceGeometry(c, t, L, L * 1e-3, np.array([0, n], dtype=np.int64), LAM, 0.1 * LAM)


def _device_rows(B, cl, name, count, dtype):
    import torch
    t = torch.empty(count, dtype=dtype, device="cuda")
    B._copy_ptr(t, getattr(cl.info(), name), count * t.element_size())
    return t


def test_neighbour_search(B):
    import torch
    n, pairs = (1 << 27) + 9, 9
    cl = B.build_cloud(_lattice(B, n, pairs), max_nnzb=n + 64)
    say(f"[many] {n} wires: {cl.nnzb} blocks, {cl.n_pairs} pairs")
    assert cl.nnzb == n + 2 * pairs and cl.n_pairs == pairs
    row_ptr = _device_rows(B, cl, "row_ptr", n + 1, torch.int64)
    deg = row_ptr[1:] - row_ptr[:-1]
    assert int((deg == 1).sum()) == n - 2 * pairs and int((deg == 2).sum()) == 2 * pairs
    diag = _device_rows(B, cl, "diag_pos", n, torch.int64)
    col = _device_rows(B, cl, "col_idx", cl.nnzb, torch.int32)
    assert bool((col[diag] == torch.arange(n, device="cuda")).all())
    B.destroy(cl)


@pytest.mark.parametrize("s,variant", [(2, -1), (1, 7)])
def test_product(B, s, variant):
    import torch
    n = (1 << 26) + 11
    cl = B.build_cloud(_lattice(B, n, 5), max_nnzb=n + 64)
    g = torch.Generator(device="cuda").manual_seed(3)
    Z = torch.view_as_complex(torch.randn((cl.nnzb, 7, 7, 2), generator=g, device="cuda"))
    X = torch.view_as_complex(torch.randn((n * 7, s, 2), generator=g, device="cuda"))
    Y = B.spmm(cl, Z, X, B.C64, variant).reshape(n, 7, s)
    rp = _device_rows(B, cl, "row_ptr", n + 1, torch.int64)
    rows = torch.cat([torch.arange(o, o + 4096, device="cuda") for o in (0, (1 << 25) - 2048, n // 2, n - 4096)])
    rows = rows[rp[rows + 1] - rp[rows] == 1]   # the wires that stand alone
    z, x = Z[rp[rows]].to(torch.complex128), X.reshape(n, 7, s)[rows].to(torch.complex128)
    ref = sum(z[:, :, k, None] * x[:, k, None, :] for k in range(7))
    size = sum(z[:, :, k, None].abs() * x[:, k, None, :].abs() for k in range(7))
    err = ((Y[rows] - ref).abs() / size).max().item()
    say(f"[many] product of {n} rows, {s} columns, variant {variant}: error {err:.1e}")
    assert err <= 32 * 2.0 ** -24
    assert int((Y.abs().amax((1, 2)) == 0).sum()) == 0
    B.destroy(cl)


def test_gradient_of_many_rows(B):
    """Weight gradients over more splits than one launch counts threads for: a batch repeated whole times
    has its own gradient; the partial sums are added one after the other in FP32, splits * eps at most."""
    import torch
    base, times = 4096, 18176
    splits = base * times // 512
    assert splits * 462 * 64 > 1 << 32
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 200 * GB:
        pytest.skip("needs 200 GB of device memory")
    g = torch.Generator(device="cuda").manual_seed(5)
    feat = torch.randn((base, 192), generator=g, device="cuda").to(torch.bfloat16).view(torch.int16)
    T = torch.randn((base, 14), generator=g, device="cuda")
    th = torch.as_tensor(W.mlp_init(7).astype(np.float32), device="cuda")
    one, loss1 = B.mlp_grad(th, feat, T)
    idx = torch.arange(base, device="cuda").repeat(times)
    many, loss = B.mlp_grad(th, feat, T, idx)
    err = ((many - one).double().norm() / one.double().norm()).item()
    say(f"[many] gradient of {base * times} rows: {err:.1e}")
    assert err <= splits * 2.0 ** -24
    assert abs(loss.item() - loss1.item()) <= 1e-5 * loss1.item()
