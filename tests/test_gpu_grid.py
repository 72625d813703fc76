"""The gridded form of the patch (many bins: spread onto a uv grid, transform)
against the FP64 oracle, at the sizes where it can go wrong: patch sizes on
both sides of each grid size, sides of very different length, even and odd,
cells of either sign, grids off the source, short last bins on both axes,
baselines of many and of few bins, windows, given factors, the normalised
patch, and bins that are not finite.

Bound: the kernel's aliasing is at most 3.8e-8 of a term per axis and its FP32
evaluation and products about 1.2e-7, so a patch is off by less than 5e-7 of
sum |c_k|; the stochastic roundings add 2^-12 sqrt(sum |c_k|^2) times about 1.5
per operand and pixel (five standard deviations are allowed)."""
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
    if name == "uniform":  # 300 bins per baseline, short last bins on both axes
        return ps.tiny_random(5, n_ant=20, n_t=301, n_ch=15, nt=3, nc=4, radius_m=3000.0, dt=8.0)
    if name == "bda":  # from 1 to 64 samples, from one bin per baseline and band to many
        return ps.tiny_random(8, n_ant=24, n_t=400, n_ch=21, nt=64, nc=8, radius_m=4000.0, dt=4.0, bda=True)
    if name == "band":  # few times, many channels: baselines of 3 x 64 bins
        return ps.tiny_random(11, n_ant=30, n_t=3, n_ch=64, nt=1, nc=1, radius_m=2000.0, dt=60.0, nu_lo=0.9e9, nu_hi=1.7e9)
    raise ValueError(name)


OBS = {}


def _case(pk, name):
    if name not in OBS:
        o = _obs(name)
        OBS[name] = (o, pk.DeviceObservation(o))
    return OBS[name]


def _src(nl, nm, r_deg=0.9, pa=0.8, cell=(CELL, CELL), off=(0.0, 0.0)):
    l0, m0 = ps.direction(r_deg * ps.DEG, pa)
    dl, dm = cell
    return ps.Source(l0=l0, m0=m0, l_first=l0 + (off[0] - 0.5 * (nl - 1)) * dl, m_first=m0 + (off[1] - 0.5 * (nm - 1)) * dm,
                     dl=dl, dm=dm, nl=nl, nm=nm)


def _bound(prec, obs, D):
    c = np.abs(obs.W * D)
    b = 5e-7 * float(np.sum(c))
    if prec in ("mixed_fp16", "sr_fp16"):
        b += 2.0 * 5.0 * 1.5 * 2.0 ** -12 * float(np.sqrt(np.sum(c * c))) * (2.0 ** 0.5 if prec == "sr_fp16" else 1.0)
    return b


# sizes at which a side changes its grid (65 | 66, 130 | 131, 261 | 262), the symmetric families' sizes, thin patches
@pytest.mark.parametrize("nl,nm", [(65, 66), (130, 131), (261, 40), (257, 257), (262, 33), (129, 129), (600, 7)])
@pytest.mark.parametrize("name", ["uniform", "bda"])
def test_sizes(pk, name, nl, nm):
    obs, dobs = _case(pk, name)
    assert obs.K >= 24576
    src = _src(nl, nm)
    D = orc.decorr(obs, src.l0, src.m0)
    ref = orc.patch_factored(obs, src, D)
    for prec in ("fp32", "split_bf16", "split_fp16"):
        P = pk.patch(dobs, src, prec=prec).double().cpu().numpy()
        e, b = float(np.max(np.abs(P - ref))), _bound(prec, obs, D)
        print(f"{name} K={obs.K} {nl}x{nm} {prec}: {e / np.max(np.abs(ref)):.2e} of the peak, {e / b:.2f} of the bound", flush=True)
        assert e <= b


@pytest.mark.parametrize("name", ["uniform", "bda", "band"])
@pytest.mark.parametrize("cell,off", [((-CELL, CELL), (0.0, 0.0)), ((CELL, -3 * CELL), (17.25, -60.5)),
                                      ((20 * CELL, 11 * CELL), (0.0, 3.0)), ((1e-3 * CELL, CELL), (0.0, 0.0))])
def test_cells_and_offsets(pk, name, cell, off):
    """Cells of either sign, from a thousandth of a beam (every bin in one
    cell) to well beyond it (positions wrap round the torus many times)."""
    obs, dobs = _case(pk, name)
    src = _src(129, 140, cell=cell, off=off)
    D = orc.decorr(obs, src.l0, src.m0)
    ref = orc.patch_factored(obs, src, D)
    P = pk.patch(dobs, src, prec="split_bf16").double().cpu().numpy()
    e, b = float(np.max(np.abs(P - ref))), _bound("split_bf16", obs, D)
    print(f"{name} cells {cell}, offset {off}: {e / b:.2f} of the bound", flush=True)
    assert e <= b


@pytest.mark.parametrize("prec", ["mixed_fp16", "sr_fp16"])
def test_stochastic_roundings(pk, prec):
    obs = ps.tiny_random(6, n_ant=26, n_t=420, n_ch=20, nt=5, nc=2, radius_m=3000.0, dt=8.0)
    assert obs.K >= 1 << 18
    dobs = pk.DeviceObservation(obs)
    src = _src(65, 65)
    D = orc.decorr(obs, src.l0, src.m0)
    ref = orc.patch_factored(obs, src, D)
    P = pk.patch(dobs, src, prec=prec)
    Q = pk.patch(dobs, src, prec=prec)
    assert torch.equal(P, Q)
    e, b = float(np.max(np.abs(P.double().cpu().numpy() - ref))), _bound(prec, obs, D)
    print(f"{prec}: {e / b:.2f} of the bound", flush=True)
    assert e <= b


def test_windows_given_factors_and_normalised(pk):
    obs, dobs = _case(pk, "uniform")
    src = _src(129, 100)
    D = orc.decorr(obs, src.l0, src.m0)
    ref = orc.patch_factored(obs, src, D)
    b = _bound("fp32", obs, D)
    given = pk.patch(dobs, src, prec="fp32", D=pk.decorr(dobs, src.l0, src.m0)).double().cpu().numpy()
    assert np.max(np.abs(given - ref)) <= b
    peak = 2.0 * float(np.sum(obs.W * D).real)
    for kw in ({}, {"D": pk.decorr(dobs, src.l0, src.m0)}):
        norm = pk.patch(dobs, src, prec="fp32", normalise=True, **kw).double().cpu().numpy()
        assert np.max(np.abs(norm - ref / peak)) <= 2 * b / abs(peak)
    win = ps.tapered_windows(obs)
    Dw = orc.decorr(win, src.l0, src.m0)
    P = pk.patch(pk.DeviceObservation(win), src, prec="fp32").double().cpu().numpy()
    assert np.max(np.abs(P - orc.patch_factored(win, src, Dw))) <= _bound("fp32", win, Dw)


def test_batched_equals_single(pk):
    """Sources of several grids in one call, each against its own call: the
    same spreading in other workgroups, so apart by rounding only."""
    obs, dobs = _case(pk, "bda")
    srcs = [_src(129, 129, pa=q) for q in (0.1, 1.7, 2.9)] + [_src(257, 257, pa=4.0), _src(100, 131, pa=5.0)]
    parts = pk.split_patches(pk.patch_batched(dobs, srcs, prec="split_fp16", normalise=True), srcs)
    for s, P in zip(srcs, parts):
        Q = pk.patch(dobs, s, prec="split_fp16", normalise=True)
        assert float((P - Q).abs().max()) <= 1e-6 * float(Q.abs().max())


def test_not_finite_and_zero_weights(pk):
    obs, _ = _case(pk, "uniform")
    src = _src(129, 129)
    import dataclasses
    for bad in (np.nan, np.inf):
        W = obs.W.copy()
        W[obs.K // 3] = bad
        P = pk.patch(pk.DeviceObservation(dataclasses.replace(obs, W=W)), src, prec="fp32")
        assert bool(torch.isnan(P).all())
    zero = pk.DeviceObservation(dataclasses.replace(obs, W=np.zeros_like(obs.W)))
    for norm in (False, True):
        assert float(pk.patch(zero, src, prec="fp32", normalise=norm).abs().max()) == 0.0
    # weights far from 1 scale the patch
    P = pk.patch(pk.DeviceObservation(obs), src, prec="split_fp16")
    for f in (2.0 ** 40, 2.0 ** -40):
        Q = pk.patch(pk.DeviceObservation(dataclasses.replace(obs, W=obs.W * np.float32(f))), src, prec="split_fp16")
        assert torch.equal(Q, P * f)


@pytest.mark.parametrize("spacing", ["even", "down", "uneven"])
@pytest.mark.parametrize("nc", [2, 3, 4, 5, 8, 16, 17])
def test_channels_per_bin(pk, nc, spacing):
    """Bins of evenly spaced channels are summed by their spacing (3 to 16
    channels, either direction), others channel by channel; short last bins on
    both axes, of one channel and of one time."""
    import dataclasses
    obs = ps.tiny_random(40 + nc, n_ant=26, n_t=76, n_ch=3 * nc + 1, nt=3, nc=nc, radius_m=1500.0, dt=10.0)
    f = np.asarray(obs.freq_hz, dtype=np.float64)
    if spacing == "down":
        f = f[::-1].copy()
    if spacing == "uneven":
        f = f + np.random.default_rng(nc).uniform(-0.3, 0.3, f.size) * abs(f[1] - f[0])
    obs = dataclasses.replace(obs, freq_hz=f)
    assert obs.K >= 24576
    dobs = pk.DeviceObservation(obs)
    src = _src(65, 100)
    D = orc.decorr(obs, src.l0, src.m0)
    ref = orc.patch_factored(obs, src, D)
    P = pk.patch(dobs, src, prec="fp32").double().cpu().numpy()
    e, b = float(np.max(np.abs(P - ref))), _bound("fp32", obs, D)
    print(f"nc {nc} {spacing} K={obs.K}: {e / np.max(np.abs(ref)):.2e} of the peak, {e / b:.2f} of the bound", flush=True)
    assert e <= b


def test_spans(pk):
    """From one span per workgroup (K / 512 of them) to four each of 768, with
    baselines that hold from none of a span's first bins to several spans."""
    for seed, n_ant, n_t, n_ch in ((1, 9, 700, 1), (2, 60, 14, 1), (3, 40, 1050, 1), (4, 4, 45000, 3)):
        obs = ps.tiny_random(seed, n_ant=n_ant, n_t=n_t, n_ch=n_ch, nt=1, nc=1, radius_m=2500.0, dt=7200.0 / n_t)
        src = _src(129, 129)  # (smaller patches of so few bins take the dense form)
        D = orc.decorr(obs, src.l0, src.m0)
        assert obs.K >= 24576
        ref = orc.patch_factored(obs, src, D)
        P = pk.patch(pk.DeviceObservation(obs), src, prec="split_bf16", normalise=True).double().cpu().numpy()
        peak = 2.0 * float(np.sum(obs.W * D).real)
        e, b = float(np.max(np.abs(P - ref / peak))), 2 * _bound("split_bf16", obs, D) / abs(peak)
        print(f"K={obs.K}, {n_ant} antennas: {e / b:.2f} of the bound", flush=True)
        assert e <= b


@pytest.mark.parametrize("n_t,n_ch,dt", [(60, 2, 600.0), (1500, 2, 25.0), (30, 64, 900.0)])
def test_sparse_tracks(pk, n_t, n_ch, dt):
    """Long baselines over a wide band in long steps: tracks that leave a tile
    within a few bins, so that windows are folded into the grid itself, and
    ones that do so in part."""
    obs = ps.tiny_random(5, n_ant=30 if n_t < 100 else 9, n_t=n_t, n_ch=n_ch, nt=1, nc=1, radius_m=6000.0, dt=dt, nu_lo=0.9e9, nu_hi=1.7e9)
    assert obs.K >= 24576
    src = _src(140, 129)
    D = orc.decorr(obs, src.l0, src.m0)
    ref = orc.patch_factored(obs, src, D)
    P = pk.patch(pk.DeviceObservation(obs), src, prec="fp32").double().cpu().numpy()
    e, b = float(np.max(np.abs(P - ref))), _bound("fp32", obs, D)
    print(f"K={obs.K}: {e / b:.2f} of the bound", flush=True)
    assert e <= b
