"""Scratch memory of the compiled kernels, from the metadata notes of the gfx950 code objects in libblink.so. Scratch
comes out of memory that the runtime allocates beside the caller's workspace (bytes per lane x 64 lanes x
every wave that can be resident: 300 MB for 1120 bytes), so the folded path's kernels, which every call
launches, keep to a few registers' worth.
"""
import os
import struct

import pytest

from paper_2505_15204_amd import build

msgpack = pytest.importorskip("msgpack")

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    at = data.find(BUNDLE)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(BUNDLE))
        p = at + len(BUNDLE) + 8
        for _ in range(n):
            off, size, k = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + k].decode()
            p += 24 + k
            if "gfx950" in triple and size:
                yield data[at + off:at + off + size]
        at = data.find(BUNDLE, p)


def kernels(elf):
    """The kernels of an ELF code object's AMDGPU metadata note (type 32)."""
    assert elf[:4] == b"\x7fELF"
    (shoff,) = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        end = off + size
        while kind == 7 and off < end:                     # SHT_NOTE
            namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (namesz + 3) // 4 * 4
            if ntype == 32 and elf[off + 12:off + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]
            off = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def scratch():
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        data = f.read()
    return {k[".name"]: k[".private_segment_fixed_size"] for elf in code_objects(data) for k in kernels(elf)}


@pytest.mark.parametrize("name,count", [("k_fold_bin", 8), ("k_fold_image", 15), ("k_fold_desc", 6)])
def test_folded_path(scratch, name, count):
    got = {k: v for k, v in scratch.items() if name in k}
    assert len(got) >= count, sorted(got)
    assert max(got.values()) <= 64, got
