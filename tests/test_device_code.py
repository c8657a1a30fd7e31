"""What the kernel descriptors of the built library ask the hardware for (LLVM's
AMDGPU code object: 64-byte descriptors at the symbols <kernel>.kd, user SGPR
requests in the 16 bits at byte 56)."""
import struct

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 32)


def descriptors(elf):
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    sec = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * shentsize) for i in range(shnum)]
    for s in sec:
        if s[1] != 11:  # SHT_DYNSYM
            continue
        strings = sec[s[6]]
        for q in range(s[4], s[4] + s[5], 24):
            name, _, _, shndx, value, size = struct.unpack_from("<IBBHQQ", elf, q)
            a = strings[4] + name
            text = elf[a:elf.index(b"\0", a)].decode()
            if text.endswith(".kd") and size == 64:
                o = sec[shndx][4] + value - sec[shndx][3]
                yield text[:-3], elf[o:o + 64]


def test_no_kernel_reads_its_dispatch_packet():
    """The packet lies in host memory.  Reading it (as the compiler does to place an
    array that is indexed at run time in LDS) costs a launch of many blocks 10 us."""
    import paper_2508_13304_amd as m
    seen, bad = 0, []
    for elf in code_objects(open(m.LIB_PATH, "rb").read()):
        for name, kd in descriptors(elf):
            seen += 1
            if struct.unpack_from("<H", kd, 56)[0] & 2:  # ENABLE_SGPR_DISPATCH_PTR
                bad.append(name)
    assert seen > 100 and not bad, (seen, bad)
