"""What the compiler made of kernels that have no register to spare, read from the built library: scratch memory per lane."""
import os
import re
import struct

import msgpack
import pytest

import paper_2405_03917_amd as cq


def _code_objects(blob):
    """The gfx950 ELF images of the library's offload bundles."""
    for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", blob):
        at = m.end()
        (n,) = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name:
                yield blob[m.start() + offset:m.start() + offset + size]


def _kernels(elf):
    """Metadata records of a code object's kernels (the msgpack note of its AMDGPU section)."""
    assert elf[:4] == b"\x7fELF"
    (shoff,) = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, _, _, offset, size = struct.unpack_from("<IQQQQ", elf, shoff + i * entry + 4)
        if kind != 7:                                   # SHT_NOTE
            continue
        name_size, desc_size, note = struct.unpack_from("<III", elf, offset)
        if note == 32:                                  # NT_AMDGPU_METADATA
            at = offset + 12 + (name_size + 3) // 4 * 4
            yield from msgpack.unpackb(elf[at:at + desc_size], strict_map_key=False)["amdhsa.kernels"]


@pytest.fixture(scope="module")
def scratch():
    with open(cq.LIB_PATH, "rb") as f:
        blob = f.read()
    return {k[".name"]: k[".private_segment_fixed_size"] for elf in _code_objects(blob) for k in _kernels(elf)}


@pytest.mark.skipif(not os.path.exists(cq.LIB_PATH), reason="library not built")
def test_four_heads_over_pre_rope_keys_leave_scratch_alone(scratch):
    """A value kept for the end of an item and spilled at its start is a load that waits for the codebooks: 192 bytes in the
    fused step of CQ-8c8b cost 2 to 5 us a call."""
    quads = {k: v for k, v in scratch.items() if "decode_quad_kernel" in k}
    assert len(quads) == 10                             # two formats x (attention, step; the same over pre-RoPE keys; layers)
    assert max(quads.values()) <= 64, quads
