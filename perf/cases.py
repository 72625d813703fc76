"""Timed cases of the distorted-PSF library: what a user's program has it do.

``listed()`` gives the cases, ``draw(rng)`` more of the same ranges,
``prepare`` the inputs and handles a program holds before a call, ``run`` one
pass through the public entry points, ``work`` the bytes and operations a
pass cannot do without and ``exact`` the same outputs in 64 bits from plain
torch.

The observations are the synthetic MeerKAT-shaped ones of the repository's
workloads (a Gaussian core and an outer annulus of antennas, Earth-rotation
tracks, uniform or baseline-dependent averaging bins), made on the GPU here
so that a case can be prepared many times.  The antenna layout follows from
the case (it fixes the number of bins); declination, hour angle, weights,
directions, cotangents and fluxes follow from the seed.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2009_07010_amd as pk

C_LIGHT = 299792458.0
OMEGA = 7.2921150e-5
ARCSEC = math.pi / (180.0 * 3600.0)
DEG = math.pi / 180.0
LATITUDE = -30.7 * DEG
DEV = "cuda"
F64 = torch.float64


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _case(name, kind, **kw):
    """A case: observation sizes, patches, arithmetic and the call."""
    c = dict(kind=kind, n_ant=64, n_t=3600, dt=2.0, n_ch=32, nu_lo=1.3e9, nu_hi=1.5e9, bin_t=10, bin_c=4,
             window=False, n_src=1, nl=257, nm=257, sizes="", cell=1.5, off_l=0.0, off_m=0.0, r_lo=0.2, r_hi=2.0,
             prec="split_bf16", normalise=False, cycles=0, grid=0)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: seven antennas, ten minutes, one channel; launches and latency only
        _case("patch_tiny", "patch", n_ant=7, n_t=600, dt=1.0, n_ch=1, nu_lo=1.4e9, nu_hi=1.4e9, bin_t=30, bin_c=1,
              nl=65, nm=65, cell=2.0, r_lo=0.3, r_hi=0.9),
        # a user's own cut-out: odd, unequal sides, the grid off the source, uneven bins, FP32 products
        _case("patch_ragged_fp32", "patch", n_ant=32, n_t=1801, n_ch=30, bin_t=0, bin_c=0, nl=150, nm=203,
              off_l=11.3, off_m=-6.7, prec="fp32"),
        # one PSF of the uniform-bin observation (K = 5.8M) in the fastest arithmetic
        _case("patch_257_sr", "patch", prec="sr_fp16"),
        # the same PSF as the precision baseline forms it, normalised at the source
        _case("patch_257_fp32_norm", "patch", prec="fp32", normalise=True),
        # the largest: sixteen directions on baseline-dependent bins (K about 2.6e8), three patch sizes
        _case("batch16_bda", "batch", n_t=14400, dt=1.0, n_ch=64, bin_t=0, bin_c=0, n_src=16, sizes="65,129,257",
              r_lo=0.05, r_hi=3.0, prec="sr_fp16"),
        # a wide band in short bins (K = 23.2M) in the binding's default arithmetic
        _case("batch_wideband", "batch", n_t=1800, n_ch=64, nu_lo=0.9e9, nu_hi=1.7e9, bin_t=5, bin_c=2, n_src=3,
              r_lo=0.1, r_hi=3.0),
        # one step of fitting sixteen positions and fluxes: forward, flux, adjoint
        _case("fit_step", "fit", n_src=16, nl=129, nm=129),
        # the adjoint alone, on a patch too large for one row range
        _case("adjoint_257", "adjoint", n_t=900, dt=4.0, bin_t=5, n_src=2, nl=257, nm=257, prec="split_fp16"),
        # deconvolution: minor cycles kept on the device, a PSF per peak
        _case("clean_257", "clean", n_t=1800, dt=4.0, cycles=6),
        # the image-plane approximation for many directions from one spectrum
        _case("method2_512", "method2", n_t=450, dt=16.0, n_ch=16, bin_t=2, bin_c=2, n_src=16, grid=512, r_hi=3.0),
        # factors of long, wide, windowed bins (20 s x 2 MHz of 1 s x 50 kHz samples)
        _case("decorr_window", "decorr", n_t=7200, dt=1.0, n_ch=120, nu_lo=1.397e9, nu_hi=1.403e9, bin_t=20,
              bin_c=40, window=True, r_lo=0.5, r_hi=4.5),
        # the patch with its exact w phase
        _case("fullw_129", "fullw", n_t=900, dt=8.0, n_ch=16, bin_t=5, bin_c=2, nl=129, nm=129, cell=3.0,
              prec="split_fp16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above (no name): sizes spread over their
    logarithm, odd ones among them."""
    kind = rng.choice(["patch", "patch", "patch", "batch", "batch", "fit", "adjoint", "clean", "method2", "decorr",
                       "fullw"])
    c = _case(None, kind)
    c["n_ant"] = _log_int(rng, 7, 64)
    c["n_t"] = _log_int(rng, 300, 3600)
    c["dt"] = round(7200.0 / c["n_t"], 3)
    c["n_ch"] = _log_int(rng, 1, 64)
    c["nu_lo"], c["nu_hi"] = rng.choice([(1.3e9, 1.5e9), (0.9e9, 1.7e9), (1.397e9, 1.403e9)])
    if rng.random() < 0.4:
        c["bin_t"], c["bin_c"] = 0, 0
    else:
        c["bin_t"], c["bin_c"] = _log_int(rng, 1, 30), min(c["n_ch"], _log_int(rng, 1, 8))
    c["prec"] = rng.choice(["split_bf16", "split_fp16", "mixed_fp16", "sr_fp16", "fp32"])
    c["cell"] = round(math.exp(rng.uniform(math.log(0.5), math.log(4.0))), 3)
    c["window"] = rng.random() < 0.2
    c["r_lo"], c["r_hi"] = 0.05, 3.0
    n = rng.choice([33, 64, 65, 100, 128, 129, 129, 200, 256, 257, 257, 300])
    c["nl"], c["nm"] = n, n if rng.random() < 0.7 else _log_int(rng, 33, 300)
    if rng.random() < 0.3:
        c["off_l"], c["off_m"] = round(rng.uniform(-20.0, 20.0), 2), round(rng.uniform(-20.0, 20.0), 2)
    if kind == "batch":
        c["n_src"] = rng.randint(2, 8)
        c["sizes"] = rng.choice(["", "65,129,257", "64,150"])
    elif kind == "fit":
        c["n_src"] = rng.randint(1, 8)
    elif kind == "adjoint":
        c["n_src"] = rng.randint(1, 3)
    elif kind == "clean":
        c["cycles"], c["off_l"], c["off_m"] = rng.randint(2, 6), 0.0, 0.0
    elif kind == "method2":
        c["n_src"], c["grid"] = rng.randint(1, 24), rng.choice([64, 256, 512])
        c["n_t"] = min(c["n_t"], 600)
    elif kind == "fullw":
        c["n_t"], c["n_ch"] = min(c["n_t"], 600), min(c["n_ch"], 16)
        c["nl"], c["nm"] = min(c["nl"], 129), min(c["nm"], 129)
    if kind == "patch" and rng.random() < 0.3:
        c["normalise"] = True
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _layout(c):
    """Antenna positions (E, N, U) in metres: a disc of 1 km for the smallest
    array, else a Gaussian core of 300 m and an annulus of 1-4 km."""
    n = c["n_ant"]
    g = np.random.default_rng(np.random.SeedSequence([29, n]))
    if n < 12:
        r, th = 1000.0 * np.sqrt(g.random(n)), 2.0 * math.pi * g.random(n)
        en = np.stack([r * np.cos(th), r * np.sin(th)], axis=1)
    else:
        n_out = n // 4
        core = g.normal(0.0, 300.0, size=(n - n_out, 2))
        r, th = np.sqrt(g.uniform(1.0e6, 1.6e7, size=n_out)), 2.0 * math.pi * g.random(n_out)
        en = np.concatenate([core, np.stack([r * np.cos(th), r * np.sin(th)], axis=1)])
    return np.concatenate([en, np.zeros((n, 1))], axis=1)


def _bins(c):
    """(baseline vectors, bin lengths per baseline, time and channel bins per baseline)."""
    pos = _layout(c)
    p, q = np.triu_indices(len(pos), k=1)
    enu = pos[q] - pos[p]
    if c["bin_t"] == 0:  # baseline-dependent: floor(B_max / |b|), 1-64 samples x 1-8 channels
        L = np.linalg.norm(enu, axis=1)
        r = np.floor(L.max() / L).astype(np.int64)
        b = np.stack([np.clip(r, 1, 64), np.clip(r, 1, 8)], axis=1)
    else:
        b = np.tile(np.array([[c["bin_t"], c["bin_c"]]], np.int64), (len(enu), 1))
    b = np.minimum(b, [[c["n_t"], c["n_ch"]]])
    n_tb, n_fb = -(-c["n_t"] // b[:, 0]), -(-c["n_ch"] // b[:, 1])
    return enu, b, n_tb, n_fb


def _tracks(xyz, ha, dec):
    """Earth-rotation uvw (metres) of baselines xyz [n, 3] at hour angles ha [n, h] or [h]."""
    X, Y, Z = (xyz[:, i:i + 1] for i in range(3))
    sh, ch = torch.sin(ha), torch.cos(ha)
    sd, cd = math.sin(dec), math.cos(dec)
    return torch.stack([X * sh + Y * ch, -X * sd * ch + Y * sd * sh + Z * cd, X * cd * ch - Y * cd * sh + Z * sd], -1)


def _frac(n, size):
    """Centre offset of each of n samples in its bin as a fraction of the bin: [n_bl, n]."""
    i = torch.arange(n, device=DEV)[None, :]
    first = (i // size[:, None]) * size[:, None]
    span = torch.minimum(size[:, None], n - first)
    return (i - first + 0.5) / span - 0.5


def _observation(c, seed):
    """The observation's arrays on the GPU (the attributes DeviceObservation reads)."""
    g = np.random.default_rng(np.random.SeedSequence([31, seed]))
    dec = (-30.0 + g.uniform(-4.0, 4.0)) * DEG
    ha0 = g.uniform(-0.05, 0.05)
    enu, b, n_tb, n_fb = _bins(c)
    e = torch.as_tensor(enu, dtype=F64, device=DEV)
    sl, cl = math.sin(LATITUDE), math.cos(LATITUDE)
    xyz = torch.stack([-e[:, 1] * sl + e[:, 2] * cl, e[:, 0], e[:, 1] * cl + e[:, 2] * sl], -1)
    n_t, n_ch, dt = c["n_t"], c["n_ch"], c["dt"]
    t0 = -0.5 * n_t * dt + 0.5 * dt
    times = t0 + torch.arange(n_t, dtype=F64, device=DEV) * dt
    o = SimpleNamespace()
    o.uvw_m = _tracks(xyz, ha0 + OMEGA * times[None, :], dec)
    step = (c["nu_hi"] - c["nu_lo"]) / n_ch
    o.freq_hz = c["nu_lo"] + (torch.arange(n_ch, dtype=F64, device=DEV) + 0.5) * step
    o.bl_bin = torch.as_tensor(b, dtype=torch.int32, device=DEV)
    off = lambda n: torch.as_tensor(np.concatenate([[0], np.cumsum(n)]), dtype=torch.int64, device=DEV)
    o.bl_koff, o.bl_tboff = off(n_tb * n_fb), off(n_tb)
    # uvw at the mean time of every time bin; the sample's own row for a bin of one sample
    cnt = torch.as_tensor(n_tb, device=DEV)
    bl = torch.repeat_interleave(torch.arange(len(b), device=DEV), cnt)
    T = torch.arange(bl.numel(), device=DEV) - o.bl_tboff[:-1][bl]
    nt = o.bl_bin[:, 0].long()[bl]
    f = T * nt
    last = torch.minimum(f + nt, torch.tensor(n_t, device=DEV)) - 1
    tc = 0.5 * (times[f] + times[last])
    uc = _tracks(xyz[bl], (ha0 + OMEGA * tc)[:, None], dec)[:, 0]
    one = (last == f)[:, None]
    o.uvw_c_m = torch.where(one, o.uvw_m.view(-1, 3)[bl * n_t + f], uc)
    K = int(o.bl_koff[-1])
    gen = torch.Generator(device=DEV).manual_seed(1000003 + seed)
    o.W = 0.5 + torch.rand(K, generator=gen, device=DEV)
    o.win_t = o.win_c = None
    if c["window"]:
        # raised-cosine windows, the stronger the longer the baseline
        a = torch.linalg.norm(e, dim=1)
        a = (a / a.max())[:, None]
        cut = lambda n, size: ((1.0 - a) + a * torch.cos(math.pi * _frac(n, size)) ** 2).float()
        o.win_t, o.win_c = cut(n_t, o.bl_bin[:, 0].long()), cut(n_ch, o.bl_bin[:, 1].long())
    return o


def _sources(c, seed):
    """Directions at r_lo .. r_hi degrees and their pixel grids."""
    g = np.random.default_rng(np.random.SeedSequence([37, seed]))
    sizes = [int(s) for s in c["sizes"].split(",")] if c["sizes"] else None
    cell = c["cell"] * ARCSEC
    out = []
    for _ in range(c["n_src"]):
        r, pa = g.uniform(c["r_lo"], c["r_hi"]) * DEG, 2.0 * math.pi * g.random()
        l0, m0 = math.sin(r) * math.sin(pa), math.sin(r) * math.cos(pa)
        nl, nm = (c["nl"], c["nm"]) if sizes is None else (sizes[len(out) % len(sizes)],) * 2
        out.append(SimpleNamespace(l0=l0, m0=m0, l_first=l0 + (c["off_l"] - 0.5 * (nl - 1)) * cell,
                                   m_first=m0 + (c["off_m"] - 0.5 * (nm - 1)) * cell, dl=cell, dm=cell, nl=nl, nm=nm))
    return out


def _cotangent(c, seed, n):
    gen = torch.Generator(device=DEV).manual_seed(2000003 + seed)
    return torch.randn(n, generator=gen, device=DEV)


def _fluxes(c, seed):
    g = np.random.default_rng(np.random.SeedSequence([41, seed]))
    return torch.as_tensor(10.0 ** g.uniform(-2.0, 0.0, c["n_src"]), dtype=torch.float32, device=DEV)


def _dirty(c, seed, src):
    """A dirty image for CLEAN: three sidelobed sources on the grid plus noise."""
    g = np.random.default_rng(np.random.SeedSequence([43, seed]))
    i = torch.arange(src.nl, dtype=F64, device=DEV)[:, None]
    j = torch.arange(src.nm, dtype=F64, device=DEV)[None, :]
    img = torch.zeros((src.nl, src.nm), dtype=F64, device=DEV)
    for f in (1.0, 0.55, 0.31):
        ci, cj = g.integers(3, src.nl - 3), g.integers(3, src.nm - 3)
        r2 = (i - ci) ** 2 + (j - cj) ** 2
        img += f * torch.exp(-r2 / 18.0) * (0.8 + 0.2 * torch.cos(0.5 * torch.sqrt(r2)))
    gen = torch.Generator(device=DEV).manual_seed(3000003 + seed)
    return (img + 0.01 * torch.randn(img.shape, generator=gen, device=DEV)).float()


def _directions(c, seed):
    return [(s.l0, s.m0) for s in _sources(c, seed)]


# duration, bandwidth and frequency of the image-plane approximation's bin
def _m2_bin(c):
    ch = (c["nu_hi"] - c["nu_lo"]) / c["n_ch"]
    return max(1, c["bin_t"]) * c["dt"], max(1, c["bin_c"]) * ch, 0.5 * (c["nu_lo"] + c["nu_hi"])


def prepare(case, seed):
    """Inputs, the observation's handle, a workspace and what a program keeps."""
    c = case
    s = SimpleNamespace(c=c, obs=pk.DeviceObservation(_observation(c, seed)), ws=pk.Workspace())
    s.src = _sources(c, seed)
    if c["kind"] in ("batch", "fit"):
        s.d_srcs = pk.device_sources(s.src)[1]
    if c["kind"] == "fit":
        s.lm = torch.tensor([[q.l0, q.m0] for q in s.src], dtype=F64, device=DEV, requires_grad=True)
        s.flux = _fluxes(c, seed).requires_grad_()
    if c["kind"] in ("fit", "adjoint"):
        s.G = _cotangent(c, seed, sum(q.nl * q.nm for q in s.src))
    if c["kind"] == "clean":
        s.dirty = _dirty(c, seed, s.src[0])
    if c["kind"] == "method2":
        s.S = pk.method2_spectrum(s.obs, c["grid"], c["cell"] * ARCSEC, c["prec"], s.ws)
        s.dirs = _directions(c, seed)
    return s


def run(s):
    """One pass through the public entry points."""
    c, kind = s.c, s.c["kind"]
    if kind == "patch":
        return pk.patch(s.obs, s.src[0], c["prec"], workspace=s.ws, normalise=c["normalise"])
    if kind == "batch":
        return pk.patch_batched(s.obs, s.src, c["prec"], workspace=s.ws, d_srcs=s.d_srcs)
    if kind == "fit":
        s.lm.grad = s.flux.grad = None
        out = pk.psf_patch_fn().apply(s.lm, s.flux, s.obs, s.src, c["prec"], s.ws, s.d_srcs)
        out.backward(s.G.view_as(out))
        return {"out": out.detach(), "lm": s.lm.grad, "flux": s.flux.grad}
    if kind == "adjoint":
        return pk.patch_backward(s.obs, s.src, s.G, c["prec"], s.ws)
    if kind == "clean":
        res = s.dirty.clone()
        comps = pk.clean_hogbom_device(s.obs, s.src[0], res, c["cycles"], 0.2, 0.0, c["prec"], s.ws)
        return (res,) + tuple(comps)
    if kind == "method2":
        return pk.method2_patches(s.S, c["cell"] * ARCSEC, s.dirs, *_m2_bin(c), workspace=s.ws)
    if kind == "decorr":
        return pk.decorr(s.obs, s.src[0].l0, s.src[0].m0)
    return pk.patch_fullw(s.obs, s.src[0], c["prec"], workspace=s.ws)[0]


def work(case):
    """Bytes: each input and output once.  Operations: about 16 per sample
    for its phase and factor, and per bin, source and axis what spreading it
    onto a grid to single precision takes (the sum over bins and pixels is a
    non-uniform Fourier transform, so bins times pixels is no bound), plus the
    transforms of the pixels."""
    c = case
    enu, b, n_tb, n_fb = _bins(c)
    K, samples = float((n_tb * n_fb).sum()), float(len(b)) * c["n_t"] * c["n_ch"]
    arrays = 24.0 * len(b) * c["n_t"] + 24.0 * float(n_tb.sum()) + 8.0 * c["n_ch"]
    if c["window"]:
        arrays += 4.0 * len(b) * (c["n_t"] + c["n_ch"])
    sizes = [int(s) for s in c["sizes"].split(",")] if c["sizes"] else None
    pix = [float(c["nl"] * c["nm"]) if sizes is None else float(sizes[q % len(sizes)] ** 2) for q in range(c["n_src"])]
    fft = sum(20.0 * p * math.log2(max(p, 2.0)) for p in pix)
    per_src = 16.0 * samples + 256.0 * K
    if c["kind"] == "decorr":
        return {"bytes": arrays + 8.0 * K, "flops": 16.0 * samples}
    if c["kind"] == "method2":
        n2 = float(c["grid"]) ** 2
        return {"bytes": 8.0 * n2 + 4.0 * n2 * c["n_src"], "flops": c["n_src"] * n2 * (40.0 + 5.0 * math.log2(n2))}
    out = 4.0 * sum(pix)
    if c["kind"] in ("patch", "batch", "fullw"):
        return {"bytes": arrays + 4.0 * K + out, "flops": c["n_src"] * per_src + fft}
    if c["kind"] == "adjoint":
        return {"bytes": arrays + 4.0 * K + out, "flops": c["n_src"] * per_src + 3.0 * fft}
    if c["kind"] == "fit":
        return {"bytes": arrays + 4.0 * K + 2.0 * out, "flops": 2.0 * c["n_src"] * per_src + 4.0 * fft}
    return {"bytes": arrays + 4.0 * K + 2.0 * out, "flops": c["cycles"] * (per_src + fft)}  # clean


# --------------------------------------------------------------------------
# 64-bit reference (plain torch)
# --------------------------------------------------------------------------
def _cis(turns):
    a = (turns - torch.round(turns)) * (2.0 * math.pi)
    return torch.complex(torch.cos(a), torch.sin(a))


def _bin_blocks(c, o, l0, m0, grad):
    """Per block of baselines with equal bins: (u, v, w in wavelengths [k], D [k],
    dD/dl0, dD/dm0 or None, the bins' indices)."""
    n0 = math.sqrt(1.0 - l0 * l0 - m0 * m0)
    L = torch.tensor([l0, m0, n0 - 1.0], dtype=F64, device=DEV)
    n_t, n_ch = c["n_t"], c["n_ch"]
    for nt, nc in sorted({tuple(r) for r in o.bl_bin.tolist()}):
        bls = torch.nonzero((o.bl_bin[:, 0] == nt) & (o.bl_bin[:, 1] == nc))[:, 0]
        n_tb, n_fb = -(-n_t // nt), -(-n_ch // nc)
        ti = torch.arange(n_tb * nt, device=DEV).view(n_tb, nt)
        ci = torch.arange(n_fb * nc, device=DEV).view(n_fb, nc)
        tm, cm = (ti < n_t).double(), (ci < n_ch).double()
        ti, ci = ti.clamp(max=n_t - 1), ci.clamp(max=n_ch - 1)
        nu = o.freq_hz[ci]
        nu_k = (nu * cm).sum(1) / cm.sum(1)
        per = max(1, 24000000 // (n_tb * nt * n_fb * nc))
        for q in range(0, len(bls), per):
            bb = bls[q:q + per]
            row = o.uvw_m[bb][:, ti]                                     # [B, n_tb, nt, 3]
            tb = (o.bl_tboff[bb][:, None] + torch.arange(n_tb, device=DEV)).view(-1)
            cen = o.uvw_c_m[tb].view(len(bb), n_tb, 3)
            A, Ak = row @ L, cen @ L
            # [B, n_tb, n_fb, nt, nc]
            phi = (A[:, :, None, :, None] * nu[None, None, :, None, :] -
                   (Ak[:, :, None] * nu_k)[..., None, None]) / C_LIGHT
            x = tm[None, :, None, :, None] * cm[None, None, :, None, :]
            if o.win_t is not None:
                x = x * o.win_t[bb].double()[:, ti][:, :, None, :, None] * \
                    o.win_c[bb].double()[:, ci][:, None, :, None, :]
            e = _cis(-phi) * x
            den = x.expand(e.shape).sum((3, 4))
            den = torch.where(den == 0, torch.inf, den)
            D = e.sum((3, 4)) / den
            dl = dm = None
            if grad:
                s = nu / C_LIGHT
                d3 = [row[..., i][:, :, None, :, None] * s[None, None, :, None, :] -
                      (cen[..., i][:, :, None] * (nu_k / C_LIGHT))[..., None, None] for i in range(3)]
                dl = (-2j * math.pi) * (e * (d3[0] - d3[2] * (l0 / n0))).sum((3, 4)) / den
                dm = (-2j * math.pi) * (e * (d3[1] - d3[2] * (m0 / n0))).sum((3, 4)) / den
            uvw = cen[:, :, None, :] * (nu_k / C_LIGHT)[None, None, :, None]
            k = (o.bl_koff[bb][:, None] + torch.arange(n_tb * n_fb, device=DEV)).view(-1)
            fl = lambda t: None if t is None else t.reshape(-1)
            yield (uvw[..., 0].reshape(-1), uvw[..., 1].reshape(-1), uvw[..., 2].reshape(-1), fl(D), fl(dl), fl(dm), k)


def _axis(f, first, step, n):
    """exp(2 pi i f (first + j step)), [len(f), n]: seeds every 16 pixels times a run of 16."""
    hi = _cis(f[:, None] * (first + 16 * step * torch.arange((n + 15) // 16, dtype=F64, device=DEV)))
    lo = _cis(f[:, None] * (step * torch.arange(16, dtype=F64, device=DEV)))
    return (hi[:, :, None] * lo[:, None, :]).reshape(len(f), -1)[:, :n]


CHUNK = 1 << 17


def _shift(u, v, w, l0, m0):
    n0 = math.sqrt(1.0 - l0 * l0 - m0 * m0)
    return u - w * (l0 / n0), v - w * (m0 / n0)


def _patch64(c, o, s, normalise=False):
    P = torch.zeros((s.nl, s.nm), dtype=F64, device=DEV)
    peak = 0.0
    for u, v, w, D, _, _, k in _bin_blocks(c, o, s.l0, s.m0, False):
        up, vp = _shift(u, v, w, s.l0, s.m0)
        cf = D * o.W[k].double()
        peak = peak + 2.0 * cf.real.sum()
        for q in range(0, len(cf), CHUNK):
            z = slice(q, q + CHUNK)
            a = _axis(up[z], s.l_first - s.l0, s.dl, s.nl) * cf[z, None]
            b = _axis(vp[z], s.m_first - s.m0, s.dm, s.nm)
            P += 2.0 * (a.real.T.contiguous() @ b.real.contiguous() - a.imag.T.contiguous() @ b.imag.contiguous())
    return P / peak if normalise else P


def _grad64(c, o, s, G):
    """(dL/dl0, dL/dm0) for L = sum G P, the grid fixed."""
    l0, m0 = s.l0, s.m0
    n0 = math.sqrt(1.0 - l0 * l0 - m0 * m0)
    G = G.view(s.nl, s.nm).double()
    x = s.l_first - l0 + s.dl * torch.arange(s.nl, dtype=F64, device=DEV)
    y = s.m_first - m0 + s.dm * torch.arange(s.nm, dtype=F64, device=DEV)
    gl = gm = 0.0
    for u, v, w, D, dDl, dDm, k in _bin_blocks(c, o, l0, m0, True):
        up, vp = _shift(u, v, w, l0, m0)
        W = o.W[k].double()
        for q in range(0, len(W), CHUNK):
            z = slice(q, q + CHUNK)
            a = _axis(up[z], s.l_first - l0, s.dl, s.nl)
            b = _axis(vp[z], s.m_first - m0, s.dm, s.nm)
            GT, yGT = G.T.contiguous(), (G * y).T.contiguous()
            t = torch.complex(b.real.contiguous() @ GT, b.imag.contiguous() @ GT)
            ty = torch.complex(b.real.contiguous() @ yGT, b.imag.contiguous() @ yGT)
            at = a * t
            H, Hx, Hy = at.sum(1), (at * x).sum(1), (a * ty).sum(1)
            cw, wz = D[z] * W[z], w[z] / n0 ** 3
            j2 = 2j * math.pi
            gl = gl + 2.0 * (W[z] * dDl[z] * H + j2 * cw * (-wz * (1 - m0 * m0) * Hx - wz * l0 * m0 * Hy -
                                                            up[z] * H)).real.sum()
            gm = gm + 2.0 * (W[z] * dDm[z] * H + j2 * cw * (-wz * l0 * m0 * Hx - wz * (1 - l0 * l0) * Hy -
                                                            vp[z] * H)).real.sum()
    return torch.stack([gl, gm])


def _fullw64(c, o, s):
    l = s.l_first + s.dl * torch.arange(s.nl, dtype=F64, device=DEV)[:, None]
    m = s.m_first + s.dm * torch.arange(s.nm, dtype=F64, device=DEV)[None, :]
    n0 = math.sqrt(1.0 - s.l0 * s.l0 - s.m0 * s.m0)
    q = (torch.sqrt(1.0 - l * l - m * m) - n0).reshape(-1)
    P = torch.zeros(s.nl * s.nm, dtype=F64, device=DEV)
    for u, v, w, D, _, _, k in _bin_blocks(c, o, s.l0, s.m0, False):
        cf = D * o.W[k].double()
        for z0 in range(0, len(cf), 4096):
            z = slice(z0, z0 + 4096)
            a = _axis(u[z], s.l_first - s.l0, s.dl, s.nl) * cf[z, None]
            b = _axis(v[z], s.m_first - s.m0, s.dm, s.nm)
            ph = w[z, None] * q * (2.0 * math.pi)  # a few radians over a patch
            ab = (a[:, :, None] * b[:, None, :]).reshape(len(a), -1)
            P += 2.0 * (ab.real * torch.cos(ph) - ab.imag * torch.sin(ph)).sum(0)
    return P.view(s.nl, s.nm)


def _clean64(c, o, s, dirty):
    res = dirty.double()
    ci, cj, amp = [], [], []
    for _ in range(c["cycles"]):
        p = int(torch.argmax(res.abs()))
        i, j = divmod(p, s.nm)
        at = SimpleNamespace(**{**vars(s), "l0": s.l_first + i * s.dl, "m0": s.m_first + j * s.dm})
        P = _patch64(c, o, at)
        a = 0.2 * res[i, j]
        res = res - a * P / P[i, j]
        ci.append(i), cj.append(j), amp.append(a)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device=DEV)
    return res, i32(ci), i32(cj), torch.stack(amp), i32([len(ci)])


def _method264(c, o, dirs):
    N, cell = c["grid"], c["cell"] * ARCSEC
    eff = SimpleNamespace(l0=0.0, m0=0.0, l_first=-(N // 2) * cell, m_first=-(N // 2) * cell, dl=cell, dm=cell, nl=N,
                          nm=N)
    S = torch.fft.fft2(torch.fft.ifftshift(_patch64(c, o, eff)))
    f = torch.fft.fftfreq(N, d=1.0 / N, dtype=F64, device=DEV) / (N * cell)
    u, v = f[:, None], f[None, :]
    dt, dnu, nu = _m2_bin(c)
    out = []
    for l0, m0 in dirs:
        hp = OMEGA * dt * (u * m0 - v * l0)
        hf = (dnu / nu) * math.hypot(l0, m0) * torch.sqrt(u * u + v * v)
        out.append(torch.fft.fftshift(torch.fft.ifft2(S * torch.sinc(hp) * torch.sinc(hf)).real))
    return torch.stack(out)


def exact(case, seed):
    """What ``run`` returns, in 64 bits; None where it would take too long."""
    c = case
    _, b, n_tb, n_fb = _bins(c)
    K = float((n_tb * n_fb).sum())
    samples = float(len(b)) * c["n_t"] * c["n_ch"]
    calls = c["cycles"] if c["kind"] == "clean" else 1 if c["kind"] == "method2" else c["n_src"]
    if c["kind"] == "fullw" and K * c["nl"] * c["nm"] > 2.0e11 or calls * (samples + 500.0 * K) > 5.0e11:
        return None
    o = _observation(c, seed)
    src = _sources(c, seed)
    kind = c["kind"]
    if kind == "patch":
        return _patch64(c, o, src[0], c["normalise"])
    if kind == "batch":
        return torch.cat([_patch64(c, o, s).reshape(-1) for s in src])
    if kind in ("fit", "adjoint"):
        G = _cotangent(c, seed, sum(s.nl * s.nm for s in src))
        parts = torch.split(G, [s.nl * s.nm for s in src])
        if kind == "adjoint":
            return torch.stack([_grad64(c, o, s, g) for s, g in zip(src, parts)])
        P = torch.stack([_patch64(c, o, s) for s in src])
        f = _fluxes(c, seed).double()
        gf = (P * G.double().view_as(P)).sum((1, 2))
        gl = torch.stack([_grad64(c, o, s, g) for s, g in zip(src, parts)]) * f[:, None]
        return {"out": P * f[:, None, None], "lm": gl, "flux": gf}
    if kind == "clean":
        return _clean64(c, o, src[0], _dirty(c, seed, src[0]))
    if kind == "method2":
        return _method264(c, o, _directions(c, seed))
    if kind == "decorr":
        D = torch.empty(int(K), dtype=torch.complex128, device=DEV)
        for blk in _bin_blocks(c, o, src[0].l0, src[0].m0, False):
            D[blk[6]] = blk[3]
        return D
    return _fullw64(c, o, src[0])
