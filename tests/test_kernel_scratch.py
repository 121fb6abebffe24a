"""Registers of the built kernels, from the code objects' own metadata: no kernel keeps values in
scratch memory."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2503_16037_amd", "libsgrt.so")
EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def kernels(path):
    """(name, scratch bytes per lane) of every kernel in the library's device code objects."""
    b = open(path, "rb").read()
    out, at = [], 0
    while (at := b.find(b"\x7fELF\x02\x01", at + 1)) >= 0:
        if struct.unpack_from("<H", b, at + 18)[0] != EM_AMDGPU:
            continue
        shoff, = struct.unpack_from("<Q", b, at + 40)
        size, count = struct.unpack_from("<HH", b, at + 58)
        for h in range(at + shoff, at + shoff + size * count, size):
            if struct.unpack_from("<I", b, h + 4)[0] != SHT_NOTE:
                continue
            off, length = struct.unpack_from("<QQ", b, h + 24)
            p, end = at + off, at + off + length
            while p < end:
                n, d, kind = struct.unpack_from("<III", b, p)
                desc = p + 12 + (n + 3) // 4 * 4
                if kind == NT_AMDGPU_METADATA and b[p + 12:p + 18] == b"AMDGPU":
                    meta = msgpack.unpackb(b[desc:desc + d])
                    out += [(k[".name"], k[".private_segment_fixed_size"]) for k in meta["amdhsa.kernels"]]
                p = desc + (d + 3) // 4 * 4
    return out


def test_no_kernel_uses_scratch():
    if not os.path.exists(LIB):
        pytest.skip("libsgrt.so is not built")
    found = kernels(LIB)
    assert len(found) > 100
    assert not {name: size for name, size in found if size}
