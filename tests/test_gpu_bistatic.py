"""The three forms of the bistatic far field (two directions per thread, one, and one over four slots of
wires), their tails, several right-hand sides and clouds, sums by groups of chunks, segments longer than a
quarter wavelength, and the error of a large cloud's pattern.

With S the sum of the pattern and A the sum of its terms' sizes, the FP64 oracle and the library are each
within 1e-12 A of S: the phases reach a few hundred radians, a rounding of them is under 1e-13, and the
sums' order is worth less.  sigma = |S|^2 / (4 pi) is then within (2 |S| d + d^2) / (4 pi), d = 2e-12 A.
"""
import numpy as np
import pytest

from oracle import mom
from paper_2410_03060_amd import workloads as W
from parity_util import say

pytestmark = pytest.mark.gpu

LAM = W.WAVELENGTH


@pytest.fixture(scope="module")
def B():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03060_amd import binding
    binding.lib()
    return binding


def _cloud(seed, n, sigma, lengths=(0.4, 0.6), n_seg=8, d_c=0.0):
    rng = np.random.default_rng(seed)
    t = rng.standard_normal((n, 3))
    t /= np.linalg.norm(t, axis=1, keepdims=True)
    return W.single_cloud(rng.standard_normal((n, 3)) * sigma * LAM, t, rng.uniform(*lengths, n) * LAM, LAM, d_c,
                          n_seg=n_seg)


def _directions(seed, m):
    rng = np.random.default_rng(seed)
    r = rng.standard_normal((m, 3))
    r /= np.linalg.norm(r, axis=1, keepdims=True)
    e = np.cross(r, rng.standard_normal((m, 3)))
    return r, e / np.linalg.norm(e, axis=1, keepdims=True)


def _currents(seed, rows, R):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((rows, R)) + 1j * rng.standard_normal((rows, R))) * 1e-3


def _several():
    cloud = W.concat_clouds([_cloud(1, 700, 8.0), _cloud(2, 1, 1.0), _cloud(3, 1300, 12.0)])
    off = cloud.cloud_off
    cloud.cloud_off = np.array([off[0], off[1], off[1], off[2], off[3]], dtype=np.int64)   # with an empty cloud
    return cloud


CASES = [  # name, cloud, directions, right-hand sides
    ("two_tail_short", lambda: _cloud(4, 2000, 15.0), 15973, 4),       # 101 directions in the last block of 512
    ("two_tail_long", lambda: _cloud(4, 2000, 15.0), 16284, 4),        # 412
    ("two_several_clouds", _several, 16001, 4),
    ("two_19", lambda: _cloud(5, 500, 8.0, n_seg=20), 16100, 4),
    ("two_long_segments", lambda: _cloud(6, 2000, 15.0, lengths=(0.4, 6.0)), 16001, 4),
    ("one", lambda: _cloud(7, 2000, 15.0), 8200, 2),
    ("one_19", lambda: _cloud(8, 500, 8.0, n_seg=20), 8449, 2),
    ("one_long_segments", lambda: _cloud(9, 1900, 15.0, lengths=(5.0, 6.0)), 8200, 2),
    ("slots", lambda: _cloud(10, 515, 9.0), 300, 3),
    ("slots_19", lambda: _cloud(11, 65, 5.0, n_seg=20), 65, 1),
    ("slots_long_segments", lambda: _cloud(12, 100, 5.0, lengths=(0.3, 6.0)), 129, 2),
    ("slots_several_clouds", _several, 63, 2),
    ("groups", lambda: _cloud(13, 17000, 25.0), 70, 1),                # 67 chunks: three groups
    ("one_wire", lambda: _cloud(14, 1, 3.0), 1, 1),
]


def _form(cloud, M, R):
    """0: two directions per thread, 1: one, 2: over slots; by the workgroups that two per thread give."""
    chunk = 256 if cloud.n_seg == 8 else 64
    n_chunks = int(sum(-(-int(k) // chunk) for k in np.diff(cloud.cloud_off)))
    wide = -(-M // 512) * n_chunks * R
    return 0 if wide >= 1024 else 1 if wide >= 256 else 2


@pytest.mark.parametrize("name,make,M,R", CASES, ids=[c[0] for c in CASES])
def test_forms(B, name, make, M, R):
    import torch
    cloud = make()
    assert _form(cloud, M, R) == {"two": 0, "one": 1 if M > 1 else 2}.get(name.split("_")[0], 2)
    r, e = _directions(21, M)
    x = _currents(22, cloud.n * (cloud.n_seg - 1), R)
    cl = B.build_cloud(cloud)
    got = B.rcs(cl, torch.as_tensor(x, device="cuda"), r, e, False).cpu().numpy()
    assert got.shape == (cloud.n_clouds, R, M) and np.isfinite(got).all()
    pick = np.unique(np.r_[0:min(M, 24), max(0, M - 24):M, np.random.default_rng(23).integers(0, M, 80)])
    worst = 0.0
    nb = cloud.n_seg - 1
    for k in range(cloud.n_clouds):
        a, b = int(cloud.cloud_off[k]), int(cloud.cloud_off[k + 1])
        if a == b:
            assert not got[k].any()
            continue
        w = mom.farfield_weights(cloud, r[pick], e[pick], cloud.n_seg)[a * nb:b * nb]
        xk = x[a * nb:b * nb]
        S = np.abs(xk.T @ w)
        d = 2e-12 * (np.abs(xk).T @ np.abs(w))
        bound = (2 * S * d + d * d) / (4 * np.pi)
        worst = max(worst, float((np.abs(got[k][:, pick] - S ** 2 / (4 * np.pi)) / bound).max()))
    say(f"[bistatic] {name}: N={cloud.n} M={M} R={R}, error / bound {worst:.2e}")
    assert worst <= 1.0


def _pattern_long(cloud, x, r, e):
    """The pattern in extended precision (64-bit significand), one direction at a time."""
    f = np.longdouble
    c, t, L = (np.asarray(v, f) for v in (cloud.center, cloud.tangent, cloud.length))
    k, nb = f(2) * f("3.14159265358979323846264338") / f(cloud.wavelength), cloud.n_seg - 1
    D, xr, xi = L / (nb + 1), *(np.asarray(v, f).reshape(cloud.n, nb) for v in (x.real, x.imag))
    out = np.empty(len(r), f)
    for m in range(len(r)):
        rm, em = r[m].astype(f), e[m].astype(f)
        b = k * (t @ rm)
        h = b * D / 2
        env = (t @ em) * D * np.where(np.abs(h) < 1e-9, f(1), np.sin(h) / np.where(h == 0, f(1), h)) ** 2
        ph = (k * (c @ rm))[:, None] + b[:, None] * (-L[:, None] / 2 + np.arange(1, nb + 1) * D[:, None])
        co, si = np.cos(ph), np.sin(ph)
        re = (env[:, None] * (xr * co - xi * si)).sum()
        im = (env[:, None] * (xr * si + xi * co)).sum()
        out[m] = (re * re + im * im) / (f(4) * f("3.14159265358979323846264338"))
    return out


def test_error_of_a_large_clouds_pattern(B):
    """Three clouds within some 60 wavelengths: the error against extended precision stays below nine
    tenths of what one double for the phase of a centre costs, as the FP64 oracle has it."""
    import torch
    if np.finfo(np.longdouble).nmant < 63:
        pytest.skip("no extended precision on this host")
    err = np.zeros(2)
    size = 0.0
    for seed in (31, 32, 33):
        cloud = _cloud(seed, 2000, 15.0)
        r, e = _directions(seed, 120)
        x = _currents(seed, cloud.n * 7, 1)
        ref = _pattern_long(cloud, x[:, 0], r, e)
        cl = B.build_cloud(cloud)
        got = B.rcs(cl, torch.as_tensor(x, device="cuda"), r, e, False).cpu().numpy()[0, 0]
        plain = mom.rcs_from_currents(cloud, x, r, e)[0]
        size += float((ref * ref).sum())
        err += [float(((v - ref) ** 2).sum()) for v in (got, plain)]
    err = np.sqrt(err / size)
    say(f"[bistatic] relative error of the pattern {err[0]:.2e}, of the FP64 oracle {err[1]:.2e}")
    assert err[0] <= 0.9 * err[1]
