"""Kernels whose speed rests on keeping their values in registers, by the resource notes of the built
library: no scratch memory (a spilled register, or an array indexed so that it lies in memory)."""
import os
import struct

import msgpack
import pytest

from paper_2406_11626_amd import ccz4

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """The metadata notes of a code object: (section headers of a 64-bit ELF)."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        if kind != 7:  # SHT_NOTE
            continue
        at, length = struct.unpack_from("<QQ", elf, shoff + i * size + 0x18)
        end = at + length
        while at + 12 <= end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3) // 4 * 4
            if note == 32:  # NT_AMDGPU_METADATA
                yield msgpack.unpackb(elf[body:body + desc], strict_map_key=False)
            at = body + (desc + 3) // 4 * 4


def _kernels():
    """Name -> metadata of every kernel of the library's gfx950 code objects."""
    if not os.path.exists(ccz4.LIB_PATH):
        pytest.skip("the library is not built")
    data = open(ccz4.LIB_PATH, "rb").read()
    out, at = {}, data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in triple:
                for md in _notes(data[at + offset:at + offset + size]):
                    for k in md["amdhsa.kernels"]:
                        out[k[".name"]] = k
        at = data.find(MAGIC, at + len(MAGIC))
    return out


@pytest.fixture(scope="module")
def kernels():
    k = _kernels()
    assert len(k) > 20
    return k


@pytest.mark.parametrize("name", ["k_fill", "k_copy_faces", "k_rk4", "k_constraints_lds", "k_regrid", "k_mlp_grad",
                                  "k_mlp_forward", "k_reconstruct_lds"])
def test_no_scratch(kernels, name):
    mine = {k: v for k, v in kernels.items() if name in k}
    assert mine
    for k, v in mine.items():
        assert (v[".private_segment_fixed_size"], v[".vgpr_spill_count"]) == (0, 0), k
