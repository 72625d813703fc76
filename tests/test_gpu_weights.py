"""Patches of many bins whose weights are far from alike, against the FP64
oracle: one or a few bins 1e2 to 1e6 times the others, log-normal weights, the
number of samples of a bin, uniform weighting (the inverse of the bins per
cell of the uv plane).  Formed from the samples, from records (windows) and
from given factors; on tracks whose bins share windows and on sparse ones,
where nearly every bin is folded alone.

Bound: a term 2 |c| is off by the kernel's aliasing and the FP32 evaluation of
its taps (1.3e-7 per axis together) and by the sums' rounding, 7e-7 of |c| at
most, where a few bins outweigh all others; products of split operands add 3 * 2^-16 (BF16)
or 3 * 2^-22 (FP16) of a term, independent from bin to bin.  So a patch is off
by less than 1e-6 sum |c_k| + 2 * 3 * 2^-p sqrt(sum |c_k|^2), whatever the
weights; D's own error, at most 5e-7 per bin (1e-6 of a term), is independent
from bin to bin too (five standard deviations)."""
import dataclasses

import numpy as np
import pytest

import oracle as orc
import psf_synth as ps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
CELL = 1.5 * ps.ARCSEC


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2009_07010_amd as pk
    pk.lib()
    return pk


def _obs(name):
    if name == "uniform":  # short last bins on both axes
        return ps.tiny_random(5, n_ant=20, n_t=301, n_ch=15, nt=3, nc=4, radius_m=3000.0, dt=8.0)
    if name == "bda":
        return ps.tiny_random(8, n_ant=14, n_t=300, n_ch=21, nt=64, nc=8, radius_m=4000.0, dt=4.0, bda=True)
    if name == "sparse":  # long baselines over a wide band in long steps
        return ps.tiny_random(5, n_ant=16, n_t=30, n_ch=64, nt=1, nc=1, radius_m=6000.0, dt=900.0, nu_lo=0.9e9, nu_hi=1.7e9)
    raise ValueError(name)


def _weights(obs, dist):
    g = np.random.default_rng(17)
    W = np.array(obs.W, np.float64)
    kind, _, arg = dist.partition(":")
    if kind == "one":
        W[obs.K // 3] *= float(arg)
    elif kind == "few":
        W[g.integers(0, obs.K, 7)] *= float(arg) * 10.0 ** g.uniform(-2.0, 0.0, 7)
    elif kind == "lognormal":
        W = np.exp(float(arg) * g.standard_normal(obs.K))
    elif kind == "samples":
        W = orc.bin_table(obs).n.astype(np.float64)
    elif kind == "uv":  # cells of one over the patch's field of view
        uv = np.floor(orc.bin_centres_lambda(obs)[:, :2] * (129 * CELL)).astype(np.int64)
        _, cell, n = np.unique(uv, axis=0, return_inverse=True, return_counts=True)
        W = 1.0 / n[cell.reshape(-1)]
    return W.astype(np.float32)


BASE = {}


def _case(name):
    if name not in BASE:
        obs = _obs(name)
        assert obs.K >= 24576
        l0, m0 = ps.direction(0.9 * ps.DEG, 0.8)
        src = ps.Source.centred(l0, m0, 129, CELL, nm=140)
        BASE[name] = (obs, src, orc.decorr(obs, l0, m0))
    return BASE[name]


def _bound(prec, W, D):
    c = np.abs(W.astype(np.float64) * D)
    per_term = {"split_bf16": 3 * 2.0 ** -16, "split_fp16": 3 * 2.0 ** -22, "fp32": 0.0}[prec]
    w2 = float(np.sqrt(np.sum(W.astype(np.float64) ** 2)))
    return 1e-6 * float(np.sum(c)) + 2.0 * per_term * float(np.sqrt(np.sum(c * c))) + 5.0 * 2.0 * 5e-7 / 3.0 * w2


DISTS = ["one:1e2", "one:1e3", "one:1e4", "one:1e5", "one:1e6", "few:1e4", "lognormal:2", "samples", "uv"]


@pytest.mark.parametrize("dist", DISTS)
@pytest.mark.parametrize("name", ["uniform", "bda", "sparse"])
def test_spread_weights(pk, name, dist):
    obs, src, D = _case(name)
    obs = dataclasses.replace(obs, W=_weights(obs, dist))
    ref = orc.patch_factored(obs, src, D)
    dobs = pk.DeviceObservation(obs)
    for prec in ("fp32", "split_fp16", "split_bf16"):
        P = pk.patch(dobs, src, prec=prec).double().cpu().numpy()
        e, b = float(np.max(np.abs(P - ref))), _bound(prec, obs.W, D)
        print(f"{name} K={obs.K} {dist} (max / mean {obs.W.max() / obs.W.mean():.1e}) {prec}: "
              f"{e / np.max(np.abs(ref)):.2e} of the peak, {e / b:.2f} of the bound", flush=True)
        assert e <= b


@pytest.mark.parametrize("dist", ["one:1e3", "one:1e5", "lognormal:2", "uv"])
def test_spread_weights_from_records(pk, dist):
    """Windowed bins and given factors: records of u', v' and c."""
    obs, src, D = _case("uniform")
    obs = dataclasses.replace(obs, W=_weights(obs, dist))
    win = ps.tapered_windows(obs)
    Dw = orc.decorr(win, src.l0, src.m0)
    for o, d, given in ((win, Dw, False), (obs, D, True)):
        ref = orc.patch_factored(o, src, d)
        dobs = pk.DeviceObservation(o)
        for prec in ("fp32", "split_fp16"):
            P = pk.patch(dobs, src, prec=prec, D=pk.decorr(dobs, src.l0, src.m0) if given else None)
            e, b = float(np.max(np.abs(P.double().cpu().numpy() - ref))), _bound(prec, o.W, d)
            print(f"{'given' if given else 'windows'} {dist} {prec}: {e / b:.2f} of the bound", flush=True)
            assert e <= b


@pytest.mark.parametrize("dist", ["one:1", "one:1e4", "lognormal:2"])
def test_strong_decorrelation(pk, dist):
    """Long bins and a far source: most |D| are small against 1."""
    obs = ps.tiny_random(9, n_ant=30, n_t=600, n_ch=32, nt=10, nc=8, radius_m=6000.0, dt=20.0, nu_lo=0.9e9, nu_hi=1.7e9)
    obs = dataclasses.replace(obs, W=_weights(obs, dist))
    assert obs.K >= 24576
    l0, m0 = ps.direction(3.0 * ps.DEG, 2.3)
    src = ps.Source.centred(l0, m0, 129, CELL, nm=140)
    D = orc.decorr(obs, l0, m0)
    assert np.median(np.abs(D)) < 0.1
    ref = orc.patch_factored(obs, src, D)
    for prec in ("fp32", "split_fp16"):
        P = pk.patch(pk.DeviceObservation(obs), src, prec=prec).double().cpu().numpy()
        e, b = float(np.max(np.abs(P - ref))), _bound(prec, obs.W, D)
        print(f"median |D| {np.median(np.abs(D)):.3f} {dist} {prec}: {e / b:.2f} of the bound", flush=True)
        assert e <= b


@pytest.mark.parametrize("dist", ["one:1e5", "lognormal:2"])
def test_spread_weights_many_bins(pk, dist):
    """K = 2.8M, at sampled pixels."""
    obs = ps.tiny_random(7, n_ant=30, n_t=800, n_ch=64, nt=4, nc=2, radius_m=2000.0, dt=2.0)
    obs = dataclasses.replace(obs, W=_weights(obs, dist))
    l0, m0 = ps.direction(1.0 * ps.DEG, 2.1)
    src = ps.Source.centred(l0, m0, 129, CELL)
    D = orc.decorr(obs, l0, m0)
    ii = np.array([64, 0, 128, 64, 64, 63, 65, 10, 100, 37])
    jj = np.array([64, 0, 128, 0, 128, 64, 64, 90, 20, 111])
    ref = orc.patch_pixels(obs, src, ii, jj, D=D)
    for prec in ("fp32", "split_fp16"):
        P = pk.patch(pk.DeviceObservation(obs), src, prec=prec).double().cpu().numpy()[ii, jj]
        e, b = float(np.max(np.abs(P - ref))), _bound(prec, obs.W, D)
        print(f"K={obs.K} {dist} {prec}: {e / b:.2f} of the bound", flush=True)
        assert e <= b
