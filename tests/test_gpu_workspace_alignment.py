"""Workspaces that begin at any 4-byte address: gridded patches, whose cells are
summed by 64-bit atomics, equal those of an aligned workspace bit for bit, and
nothing is written outside the bytes given."""
import pytest

import psf_synth as ps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
GUARD = 256


@pytest.fixture(scope="module")
def pk():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_2009_07010_amd as pk
    pk.lib()
    return pk


@pytest.mark.parametrize("shift", [4, 8, 12])
def test_unaligned_workspace(pk, shift):
    obs = ps.tiny_random(5, n_ant=20, n_t=301, n_ch=15, nt=3, nc=4, radius_m=3000.0, dt=8.0)
    assert obs.K >= 24576
    dobs = pk.DeviceObservation(obs)
    srcs = []
    for q in range(3):
        l0, m0 = ps.direction(0.9 * ps.DEG, 0.8 + q)
        srcs.append(ps.Source.centred(l0, m0, 150, 1.5 * ps.ARCSEC))
    _, d = pk.device_sources(srcs)
    want = pk.patch(dobs, srcs[0], prec="fp32"), pk.patch_batched(dobs, srcs, prec="fp32")
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream().cuda_stream
    for one in (True, False):
        use = srcs[:1] if one else srcs
        need = pk.psf_workspace_bytes(dobs.struct, pk.src_array(use), "fp32")
        buf = torch.full((need + 2 * GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
        ws = buf.data_ptr() + GUARD + shift - 16
        out = torch.zeros_like(want[0] if one else want[1])
        print(f"shift {shift}, {'one' if one else 'batched'}", flush=True)
        if one:
            pk.psf_patch(dobs.struct, pk.make_src(srcs[0]), None, "fp32", out.data_ptr(), ws, need, stream)
        else:
            pk.psf_patch_batched(dobs.struct, pk.src_array(use), d.data_ptr(), "fp32", None, out.data_ptr(), ws, need, stream)
        torch.cuda.synchronize()
        assert torch.equal(out, want[0] if one else want[1])
        assert bool((buf[:GUARD + shift - 16] == 0xA5).all()) and bool((buf[GUARD + shift - 16 + need:] == 0xA5).all())
