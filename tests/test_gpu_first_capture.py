"""A program whose first launch of a kernel is a captured one: gridded patches
in every arithmetic, windowed factors and the adjoint recorded into graphs by a
fresh process, before any eager call, then replayed (with eager work and
synchronisations between the replays) and compared with eager calls."""
import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import torch
import paper_2009_07010_amd as pk
import psf_synth as ps

obs = ps.tiny_random(6, n_ant=26, n_t=420, n_ch=20, nt=5, nc=2, radius_m=3000.0, dt=8.0)
assert obs.K >= 1 << 18
wide = ps.tapered_windows(ps.tiny_random(7, n_ant=26, n_t=1200, n_ch=80, nt=20, nc=40, radius_m=3000.0, dt=1.0))
dobs, dwide = pk.DeviceObservation(obs), pk.DeviceObservation(wide)
assert wide.K >= 32768  # one lane per bin
l0, m0 = ps.direction(0.9 * ps.DEG, 0.8)
src = ps.Source.centred(l0, m0, 129, 1.5 * ps.ARCSEC)
srcs, d = pk.device_sources([src])
G = torch.randn(src.nl * src.nm, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
calls = {}
for prec in ("fp32", "split_bf16", "split_fp16", "mixed_fp16", "sr_fp16"):
    ws = pk.Workspace()
    ws.get(pk.workspace_bytes(dobs, [src], prec))
    out = torch.zeros(src.nl * src.nm, device="cuda")
    calls["patch " + prec] = (out, lambda p=prec, w=ws, o=out: pk.patch(dobs, src, prec=p, workspace=w, out=o.view(src.nl, src.nm)))
out = torch.zeros(wide.K, 2, device="cuda")
calls["windowed factors"] = (out, lambda o=out: pk.decorr(dwide, l0, m0, out=o))
for prec in ("fp32", "split_bf16", "split_fp16"):
    ws = pk.Workspace()
    ws.get(pk.workspace_bytes(dobs, [src], prec))
    out = torch.zeros(1, 2, dtype=torch.float64, device="cuda")
    calls["adjoint " + prec] = (out, lambda p=prec, w=ws, o=out: pk.patch_backward(dobs, [src], G, p, w, out=o))
torch.cuda.synchronize()
graphs = {}
for name, (out, call) in calls.items():
    print("capture", name, flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    graphs[name] = g
got = {}
for name, g in graphs.items():
    print("replay", name, flush=True)
    for rep in range(3):
        calls[name][0].zero_()
        g.replay()
        torch.cuda.synchronize()
        got.setdefault(name, []).append(calls[name][0].clone())
        torch.randn(1 << 16, device="cuda").sum().item()
for name, (out, call) in calls.items():
    out.zero_()
    call()
    torch.cuda.synchronize()
    assert out.abs().max() > 0, name
    for rep in range(3):
        assert torch.equal(got[name][rep], out), (name, rep)
print("DONE")
"""


def test_first_launch_captured():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    p = subprocess.run([sys.executable, "-u", "-c", PROGRAM], cwd=ROOT, capture_output=True, text=True, timeout=100)
    print(p.stdout, p.stderr[-2000:], flush=True)
    assert p.returncode == 0 and "DONE" in p.stdout
