"""Register and scratch use of the built kernels, read from the metadata of the
code objects in libtpfdm.so (no GPU): the single-launch kernels inline every
degree's body, so a body that grows shows there first."""
import struct

import msgpack

from paper_2609_04534_amd import tpfdm

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The device ELF images of the offload bundles in blob."""
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + n]
            p += 24 + n
            if name.startswith(b"hip") and size > 0:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, p)


def _metadata(elf):
    """The kernels' metadata maps (note type 32, name AMDGPU)."""
    assert elf[:4] == b"\x7fELF"
    phoff, = struct.unpack_from("<Q", elf, 32)
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
        end = off + size
        while kind == 4 and off < end:   # PT_NOTE
            n, d, t = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (n + 3) // 4 * 4
            if t == 32:
                yield from msgpack.unpackb(elf[desc:desc + d])["amdhsa.kernels"]
            off = desc + (d + 3) // 4 * 4


def kernels():
    with open(tpfdm.LIB_PATH, "rb") as f:
        blob = f.read()
    return {k[".name"]: k for elf in _code_objects(blob) for k in _metadata(elf)}


def test_single_launch_kernels_use_no_scratch():
    found = {n: k for n, k in kernels().items() if "k_persist_" in n}
    assert len(found) == 12   # apply, inverse and solve, four types each
    spilled = {n: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for n, k in found.items()
               if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert spilled == {}


def test_single_launch_solves_reach_three_waves_per_simd():
    """512 registers a lane and SIMD: three waves need at most 168 each."""
    regs = {n: k[".vgpr_count"] for n, k in kernels().items() if "k_persist_solve" in n}
    assert len(regs) == 4 and max(regs.values()) <= 168, regs
