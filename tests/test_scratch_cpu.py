"""Per-lane scratch memory of the built kernels, read from the code object's
metadata: a kernel that spills registers needs an eager launch before it can
be captured into a graph (the runtime allocates its scratch then), so none of
them does but those named here."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")
from paper_2009_07010_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
# the negative control, and CLEAN's peak search
SPILLS = ("k_patchILi3E", "k_absmax_")


def _metadata(elf):
    """amdhsa metadata of a code object: the descriptor of its note."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, num = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        if kind == 7:  # SHT_NOTE
            off, = struct.unpack_from("<Q", elf, shoff + i * size + 24)
            n_name, n_desc, _ = struct.unpack_from("<III", elf, off)
            return msgpack.unpackb(elf[off + 12 + (n_name + 3) // 4 * 4:][:n_desc], raw=False)
    raise AssertionError("no metadata note")


def _kernels():
    data, at, out = open(build.LIB, "rb").read(), 0, {}
    while (at := data.find(MAGIC, at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, n_id = struct.unpack_from("<QQQ", data, p)
            if size and build.ARCH in data[p + 24:p + 24 + n_id].decode():
                out.update({k[".name"]: k for k in _metadata(data[at + off:at + off + size])["amdhsa.kernels"]})
            p += 24 + n_id
        at += len(MAGIC)
    return out


def test_kernels_need_no_scratch_memory():
    if not os.path.exists(build.LIB):
        pytest.skip("library not built")
    kernels = _kernels()
    assert any("k_grid_spread" in k for k in kernels) and any("k_adjoint" in k for k in kernels)
    spills = {k: m[".private_segment_fixed_size"] for k, m in kernels.items() if m[".private_segment_fixed_size"]}
    assert not {k: v for k, v in spills.items() if not any(s in k for s in SPILLS)}
