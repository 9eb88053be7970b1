"""The counting kernels' register use, read from the built library's code object metadata (no GPU).

A SIMD holds 512 / (vector registers, rounded up to 8) wavefronts, 8 at most, and 800 / (scalar registers,
rounded up to 16, plus 16).  The comments beside the kernels say how many each was measured with; a
change elsewhere in the file that costs one of them shows here.
"""
import os
import struct

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2302_09247_amd", "libfastcod.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """Every gfx950 ELF of the bundles in a shared library."""
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def _kernels(elf):
    """Kernel entries of an AMDGPU ELF's metadata note (type 32, msgpack)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for k in range(shnum):
        typ, = struct.unpack_from("<I", elf, shoff + k * shentsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + k * shentsize + 24)
        if typ != 7:   # SHT_NOTE
            continue
        p = off
        while p < off + size:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
            d = p + 12 + (namesz + 3) // 4 * 4
            if ntype == 32:
                yield from msgpack.unpackb(elf[d:d + descsz], raw=False, strict_map_key=False).get("amdhsa.kernels", [])
            p = d + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    out = {}
    for elf in _code_objects(open(LIB, "rb").read()):
        for k in _kernels(elf):
            out[k[".name"]] = k
    assert out
    return out


def _waves(k):
    vgprs = max(1, (k[".vgpr_count"] + 7) // 8 * 8)
    sgprs = (k[".sgpr_count"] + 15) // 16 * 16 + 16
    return min(8, 512 // vgprs, 800 // sgprs)


@pytest.mark.parametrize("part,waves", [("k_count_stream_up", 6), ("k_count_stream2", 8), ("k_count_stream4", 6),
                                        ("k_count_batched", 6), ("k_pair_sort", 8)])
def test_wavefronts_per_simd(kernels, part, waves):
    found = [k for name, k in kernels.items() if part in name]
    assert found
    for k in found:
        assert k[".vgpr_spill_count"] == 0, k[".name"]
        assert _waves(k) >= waves, (k[".name"], k[".vgpr_count"], k[".sgpr_count"])
