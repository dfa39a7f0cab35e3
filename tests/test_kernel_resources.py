"""Scratch memory of the built kernels, from the metadata in the library's own code objects.

The N_g = 8 source-to-target kernels keep everything on the CU: an earlier version of theirs, whose line
buffer was in device memory and which spilled registers, ended in a fault whose cause was not shown."""
import os
import struct

import msgpack

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_1906_10734_amd", "libhpm.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
NT_AMDGPU_METADATA = 32


def _code_objects(blob):
    """The GPU ELF images of every offload bundle in the file."""
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        q = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, q)
            if b"gfx" in blob[q + 24:q + 24 + n] and size:
                yield blob[at + off:at + off + size]
            q += 24 + n
        at = blob.find(MAGIC, q)


def _kernels(elf):
    """Kernel name -> metadata of one ELF image, from its notes."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for s in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + s * shentsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + s * shentsize + 24)
        q = off
        while kind == 7 and q < off + size:  # SHT_NOTE
            namesz, descsz, note = struct.unpack_from("<III", elf, q)
            desc = q + 12 + (namesz + 3) // 4 * 4
            if note == NT_AMDGPU_METADATA:
                for k in msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]:
                    yield k[".name"], k
            q = desc + (descsz + 3) // 4 * 4


def _library():
    with open(LIB, "rb") as f:
        blob = f.read()
    return {name: k for elf in _code_objects(blob) for name, k in _kernels(elf)}


def test_ng8_kernels_use_no_scratch():
    kernels = _library()
    assert len(kernels) > 100
    ng8 = {n: k for n, k in kernels.items() if "10k_m2l_slabI" in n and "Li8E" in n}
    assert len(ng8) == 2  # FP32 and FP64
    for name, k in ng8.items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name
