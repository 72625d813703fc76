"""psf_autotune where some sources of a tile family run gridded and some dense:
the family's entry comes from a dense one, and a family that only runs gridded
is entered with what an untuned dense call takes."""
import json

import pytest

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


def _sources(sizes):
    out = []
    for q, n in enumerate(sizes):
        l0, m0 = ps.direction(0.9 * ps.DEG, 0.8 + q)
        out.append(ps.Source.centred(l0, m0, n, 1.5 * ps.ARCSEC))
    return out


def test_representatives(pk):
    obs = ps.tiny_random(9, n_ant=20, n_t=204, n_ch=16, nt=3, nc=4, radius_m=3000.0, dt=30.0)
    assert obs.K == 51680  # of 200 x 200 pixels gridded, of 33 x 33 dense
    dobs = pk.DeviceObservation(obs)
    fam = lambda f: tuple(f[k] for k in ("tbi0", "tbi1", "tbj0", "tbj1", "sym"))
    alone = {n: json.loads(pk.autotune(dobs, _sources([n]), prec="split_bf16"))["families"] for n in (33, 200)}
    assert fam(alone[33][0]) == fam(alone[200][0])
    for sizes in ([200, 33], [33, 200], [200, 33, 200]):
        doc = json.loads(pk.autotune(dobs, _sources(sizes), prec="split_bf16"))["families"]
        assert [f["nl"] for f in doc] == [33], sizes
    obs = ps.tiny_random(6, n_ant=26, n_t=420, n_ch=20, nt=5, nc=2, radius_m=3000.0, dt=8.0)
    assert obs.K >= 1 << 18  # every size gridded
    doc = json.loads(pk.autotune(pk.DeviceObservation(obs), _sources([65, 129, 257]), prec="sr_fp16"))["families"]
    assert {f["nl"]: (f["items_per_cu"], f["flush"]) for f in doc} == {65: (4, 128), 129: (1, 128), 257: (1, 128)}
    assert all(f["ms"] > 0 for f in doc)
