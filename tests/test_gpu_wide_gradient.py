"""The gradient of patches wider than the reverse-mode kernel takes (more than
288 columns) where there are bins enough that its five derivative patches run
gridded, against 64-bit sums, with weights alike and far from it.

Bound: the patch of coefficients e_k is off by at most 1e-6 sqrt(sum |e|^2)
(taps, 1.3e-7 per axis and bin, independent; five standard deviations) and 1e-7
sum |e| (rounding of the sums), and in split-BF16 by 2 * 3 * 2^-16 sqrt(sum
|e|^2); these errors meet the cotangent incoherently, so the gradient is off by
that times its norm."""
import dataclasses

import numpy as np
import pytest

import oracle as orc
import psf_synth as ps
from oracle import psf64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2009_07010_amd as pk
    pk.lib()
    return pk


@pytest.fixture(scope="module")
def case():
    obs = ps.tiny_random(9, n_ant=20, n_t=602, n_ch=15, nt=3, nc=4, radius_m=3000.0, dt=12.0)
    assert obs.K >= 150000
    l0, m0 = ps.direction(0.9 * ps.DEG, 0.8)
    cell = 1.5 * ps.ARCSEC
    src = ps.Source(l0=l0, m0=m0, l_first=l0 - 29.0 * cell, m_first=m0 - 161.5 * cell, dl=cell, dm=cell, nl=64, nm=300)
    G = np.random.default_rng(3).standard_normal((src.nl, src.nm)).astype(np.float32)
    return obs, src, G, orc.decorr_with_grad(obs, l0, m0)


def _gradient(obs, src, G, D, dDl, dDm):
    """dL/d(l0, m0) of L = sum G P in 64 bits, and the norms of its bound."""
    l0, m0 = src.l0, src.m0
    n0 = np.sqrt(1.0 - l0 * l0 - m0 * m0)
    uk = orc.bin_centres_lambda(obs)
    up, vp = psf64.wshift(uk, l0, m0)
    w = uk[:, 2] / n0 ** 3
    x, y = psf64.pixel_offsets(src)
    W = obs.W.astype(np.float64)
    c = W * D
    j2 = 2j * np.pi
    e = [W * dDl - j2 * up * c, W * dDm - j2 * vp * c, -j2 * w * (1 - m0 * m0) * c, -j2 * w * l0 * m0 * c,
         -j2 * w * (1 - l0 * l0) * c]
    H = np.zeros((3, obs.K), complex)
    for k in range(0, obs.K, 8192):
        z = slice(k, k + 8192)
        a, b = np.exp(j2 * np.outer(up[z], x)), np.exp(j2 * np.outer(vp[z], y))
        t, ty = b @ G.T.astype(np.float64), (b * y) @ G.T.astype(np.float64)
        H[0, z], H[1, z], H[2, z] = (a * t).sum(1), (a * x * t).sum(1), (a * ty).sum(1)
    g = np.array([2.0 * np.sum(e[0] * H[0] + e[2] * H[1] + e[3] * H[2]).real,
                  2.0 * np.sum(e[1] * H[0] + e[3] * H[1] + e[4] * H[2]).real])
    norms = [np.linalg.norm(G), np.linalg.norm(x[:, None] * G), np.linalg.norm(G * y)]
    root = lambda i, j: np.linalg.norm(e[i]) * norms[j]
    total = lambda i, j: np.abs(e[i]).sum() * norms[j]
    return g, [(f(0, 0) + f(2, 1) + f(3, 2), f(1, 0) + f(3, 1) + f(4, 2)) for f in (root, total)]


@pytest.mark.parametrize("ratio", [1.0, 1e3, 1e5])
def test_wide_gradient_gridded(pk, case, ratio):
    obs, src, G, (D, dDl, dDm) = case
    W = obs.W.copy()
    W[obs.K // 3] *= ratio
    obs = dataclasses.replace(obs, W=W)
    g, (root, total) = _gradient(obs, src, G, D, dDl, dDm)
    dobs = pk.DeviceObservation(obs)
    for prec in ("fp32", "split_fp16", "split_bf16"):
        got = pk.patch_backward(dobs, [src], torch.as_tensor(G.reshape(-1), device="cuda"), prec).cpu().numpy()[0]
        for i in (0, 1):
            b = 1e-6 * root[i] + 1e-7 * total[i] + (6.0 * 2.0 ** -16 * root[i] if prec == "split_bf16" else 0.0)
            e = abs(got[i] - g[i])
            print(f"K={obs.K} ratio {ratio:.0e} {prec} axis {i}: {e / np.max(np.abs(g)):.1e} of the gradient, "
                  f"{e / b:.2f} of the bound", flush=True)
            assert e <= b
