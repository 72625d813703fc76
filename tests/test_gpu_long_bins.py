"""Gridded patches of long or wide bins, whose factors are formed while
spreading or before it, on both sides of each limit of that choice: time
samples per bin (more than the spreading kernel's table holds among them),
frequency bins per time bin, channels per bin.  Against the FP64 oracle: within
5e-7 of sum |c| as other gridded patches in FP32."""
import numpy as np
import pytest

import oracle as orc
import psf_synth as ps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2009_07010_amd as pk
    pk.lib()
    return pk


# antennas, time bins, samples and channels of a bin, frequency bins
@pytest.mark.parametrize("n_ant,n_tb,nt,nc,nf", [(30, 120, 8, 1, 1), (30, 120, 12, 1, 1), (30, 60, 16, 1, 4), (30, 60, 64, 1, 2),
                                                 (30, 40, 32, 4, 6), (30, 40, 64, 4, 6), (30, 30, 2, 20, 5), (30, 30, 4, 20, 5),
                                                 (30, 30, 4, 16, 5), (30, 30, 4, 17, 5), (12, 47, 1100, 1, 12)])
def test_long_and_wide_bins(pk, n_ant, n_tb, nt, nc, nf):
    obs = ps.tiny_random(50 + nt, n_ant=n_ant, n_t=n_tb * nt - nt // 3, n_ch=nf * nc - nc // 3, nt=nt, nc=nc, radius_m=1500.0,
                         dt=7200.0 / (n_tb * nt))
    assert obs.K >= 24576
    l0, m0 = ps.direction(0.9 * ps.DEG, 0.8)
    cell = 1.5 * ps.ARCSEC
    src = ps.Source(l0=l0, m0=m0, l_first=l0 - 74.5 * cell, m_first=m0 - 100.0 * cell, dl=cell, dm=cell, nl=150, nm=201)
    D = orc.decorr(obs, l0, m0)
    ref = orc.patch_factored(obs, src, D)
    b = 5e-7 * float(np.sum(np.abs(obs.W * D)))
    dobs = pk.DeviceObservation(obs)
    for normalise in (False, True):
        P = pk.patch(dobs, src, prec="fp32", normalise=normalise).double().cpu().numpy()
        peak = 2.0 * float(np.sum(obs.W * D).real) if normalise else 1.0
        e = float(np.max(np.abs(P * peak - ref)))
        print(f"K={obs.K} bins of {nt} x {nc}, {nf} of them in frequency: {e / b:.2f} of the bound", flush=True)
        assert e <= 2 * b if normalise else e <= b
