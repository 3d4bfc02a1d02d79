"""Registers of the kernels as the compiler reports them in the built library.  No GPU needed."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_03295_amd", "libpop.so")


def kernels():
    """Metadata of every gfx950 kernel: the amdhsa notes of the code objects that the library embeds."""
    blob = open(LIB, "rb").read()
    found, at = [], blob.find(b"\x7fELF", 4)
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:                     # EM_AMDGPU
            shoff, (shentsize, shnum) = struct.unpack_from("<Q", blob, at + 40)[0], struct.unpack_from("<HH", blob, at + 58)
            for i in range(shnum):
                kind, _, _, off, size = struct.unpack_from("<IQQQQ", blob, at + shoff + i * shentsize + 4)
                if kind != 7:                                                     # SHT_NOTE
                    continue
                name, desc, note = struct.unpack_from("<III", blob, at + off)
                if note == 32:                                                    # NT_AMDGPU_METADATA
                    start = at + off + 12 + (name + 3) // 4 * 4
                    found += msgpack.unpackb(blob[start:start + desc], strict_map_key=False)["amdhsa.kernels"]
        at = blob.find(b"\x7fELF", at + 4)
    return found


def test_no_kernel_works_from_scratch_memory():
    """A register more or less spilled outside a loop is nothing (one value: 8 bytes with alignment); values that a loop reads back
    are (decode attention over an 8-bit cache, 52 bytes a lane: a step of one long sequence 3 to 5 % slower)."""
    if not os.path.exists(LIB):
        pytest.skip("libpop.so not built")
    ks = kernels()
    assert len(ks) > 100 and any("attn_decode_split_kernel" in k[".name"] for k in ks)
    assert {k[".name"]: k[".private_segment_fixed_size"] for k in ks if k[".private_segment_fixed_size"] > 8} == {}
