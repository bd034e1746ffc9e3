"""What the built device code says of itself (no GPU needed): kernels keep their registers, and hand-written instructions declare
what they change."""
import glob
import os
import re
import struct

import msgpack

import paper_2412_02252_amd as pod

CSRC = os.path.join(os.path.dirname(os.path.abspath(pod.__file__)), "csrc")


def code_objects(blob):
    """The gfx950 ELF images of the offload bundles inside the library."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        pos = at + len(magic)
        (count,) = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", blob, pos)
            target = blob[pos + 24: pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in target and size:
                yield blob[at + off: at + off + size]
        at = pos


def kernels(elf):
    """The kernels' metadata (note of type 32, MessagePack) of one code object."""
    assert elf[:4] == b"\x7fELF"
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        end = off + size
        while kind == 7 and off < end:                      # SHT_NOTE
            namesz, descsz, typ = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (namesz + 3) // 4 * 4
            if typ == 32:
                yield from msgpack.unpackb(elf[desc: desc + descsz])["amdhsa.kernels"]
            off = desc + (descsz + 3) // 4 * 4


def test_no_kernel_spills_vector_registers_or_uses_scratch_memory():
    found = [k for elf in code_objects(open(pod.lib_path(), "rb").read()) for k in kernels(elf)]
    names = [k[".name"] for k in found]
    assert any("prefill_kernel" in n for n in names) and any("decode_even_kernel" in n for n in names) and len(found) > 60
    bad = [(k[".name"], k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in found
           if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]]
    assert not bad, bad


def test_instructions_that_write_m0_say_so():
    """M0 is the compiler's to use between two statements: one that changes it names it among what it clobbers."""
    seen = 0
    for f in glob.glob(os.path.join(CSRC, "*")):
        for stmt in re.findall(r"\basm\s*(?:volatile)?\s*\((.*?)\)\s*;", open(f).read(), re.S):
            if re.search(r"\b[sv]_\w+\s+m0\b", stmt):
                seen += 1
                clobbers = stmt.split(":")[-1]
                assert '"m0"' in clobbers, (os.path.basename(f), stmt)
    assert seen
