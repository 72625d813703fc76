"""A bin that is not finite makes every pixel of a gridded patch NaN, in every
arithmetic: NaN and infinite weights, samples, bin centres and given factors,
formed from the samples, from records (windows) and from given factors."""
import dataclasses

import numpy as np
import pytest

import psf_synth as ps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
PRECS = ["fp32", "split_bf16", "split_fp16", "mixed_fp16", "sr_fp16"]


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2009_07010_amd as pk
    pk.lib()
    return pk


@pytest.fixture(scope="module")
def base():
    obs = ps.tiny_random(6, n_ant=26, n_t=420, n_ch=20, nt=5, nc=2, radius_m=3000.0, dt=8.0)
    assert obs.K >= 1 << 18
    l0, m0 = ps.direction(0.9 * ps.DEG, 0.8)
    return obs, ps.Source.centred(l0, m0, 129, 1.5 * ps.ARCSEC)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("prec", PRECS)
def test_not_finite(pk, base, prec, bad):
    obs, src = base
    W, uvw, cen = obs.W.copy(), obs.uvw_m.copy(), obs.uvw_c_m.copy()
    W[obs.K // 3] = bad
    uvw[7, 100, 1] = bad
    cen[1234, 0] = bad
    for what, o in (("weight", dataclasses.replace(obs, W=W)), ("sample", dataclasses.replace(obs, uvw_m=uvw)),
                    ("centre", dataclasses.replace(obs, uvw_c_m=cen)),
                    ("windowed weight", ps.tapered_windows(dataclasses.replace(obs, W=W))),
                    ("windowed centre", ps.tapered_windows(dataclasses.replace(obs, uvw_c_m=cen)))):
        print(f"{prec} {what} {bad}", flush=True)
        P = pk.patch(pk.DeviceObservation(o), src, prec=prec)
        assert bool(torch.isnan(P).all()), what
    dobs = pk.DeviceObservation(obs)
    D = pk.decorr(dobs, src.l0, src.m0)
    for part in (0, 1):
        d = torch.view_as_real(D).clone()
        d[obs.K // 2, part] = bad
        print(f"{prec} factor {part} {bad}", flush=True)
        assert bool(torch.isnan(pk.patch(dobs, src, prec=prec, D=torch.view_as_complex(d))).all())
    # and nothing of it is left for the next call
    assert bool(torch.isfinite(pk.patch(dobs, src, prec=prec)).all())
