"""Host-only: no kernel of the built library uses scratch memory.  The streaming loops count the vector loads in flight; a
spilled register's reload shares that counter and would make every wait one for all loads.  (The one-launch layer kernel's
widest instances keep one register there, outside their loop.)"""
import os
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_09983_amd", "libmoe_spac.so")


def _code_objects(data):
    """The gfx950 code objects of every offload bundle in the library's fat binary section."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n if n < 16 else 0):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24: p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name:
                yield data[at + off: at + off + size]
        at += len(magic)


def _kernels(elf):
    """The kernels' entries of a code object's metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entsize, num = struct.unpack_from("<HH", elf, 58)
    for i in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        if kind != 7:   # notes
            continue
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 24)
        namesz, descsz, typ = struct.unpack_from("<III", elf, off)
        if typ == 32:
            start = off + 12 + (namesz + 3) // 4 * 4
            yield from msgpack.unpackb(elf[start: start + descsz], strict_map_key=False)["amdhsa.kernels"]


def test_no_kernel_uses_scratch_memory():
    if not os.path.exists(LIB):
        pytest.fail(f"{LIB} not built (run __graft_entry__.build())")
    with open(LIB, "rb") as f:
        data = f.read()
    seen = [k for elf in _code_objects(data) for k in _kernels(elf)]
    names = " ".join(k[".name"] for k in seen)
    for n in ("stream_kernel", "routed_stream_kernel", "wide_kernel", "layer_kernel", "ffn_kernel", "route_kernel", "plan_kernel"):
        assert n in names, n
    scratch = {k[".name"]: k[".private_segment_fixed_size"] for k in seen if k[".private_segment_fixed_size"]}
    assert all("layer_kernelILi4E" in name and size <= 8 for name, size in scratch.items()), scratch
