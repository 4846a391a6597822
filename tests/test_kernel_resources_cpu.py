"""Registers of the built kernels, from the metadata of the library's own code
objects (no GPU): the forward and gradient kernels of one channel tile keep
four waves a SIMD."""
import re
import struct

import msgpack

from paper_2301_09266_amd import finc

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
NT_AMDGPU_METADATA = 32


def code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the library."""
    for m in re.finditer(MAGIC, blob):
        at = m.end()
        (n,) = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, at)
            triple = blob[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" in triple and size:
                yield blob[m.start() + off:m.start() + off + size]


def kernels():
    """name -> metadata of every kernel in the library."""
    out = {}
    for elf in code_objects(open(finc.LIB_PATH, "rb").read()):
        phoff, = struct.unpack_from("<Q", elf, 32)
        phsize, phnum = struct.unpack_from("<HH", elf, 54)
        for i in range(phnum):
            ptype, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
            end = off + size
            while ptype == 4 and off < end:   # PT_NOTE
                namesz, descsz, kind = struct.unpack_from("<III", elf, off)
                desc = off + 12 + -(-namesz // 4) * 4
                if kind == NT_AMDGPU_METADATA:
                    meta = msgpack.unpackb(elf[desc:desc + descsz])
                    out.update((k[".name"], k) for k in meta.get("amdhsa.kernels", []))
                off = desc + -(-descsz // 4) * 4
    return out


def waves(meta):
    """Waves a SIMD that the registers allow (512 a lane, in steps of eight)."""
    return 512 // max(8, -(-meta[".vgpr_count"] // 8) * 8)


def test_forward_and_gradient_waves():
    ks = kernels()
    fwd = {n: k for n, k in ks.items() if "14forward_kernelI" in n}
    grad = {n: k for n, k in ks.items() if "11grad_kernelI" in n}
    assert len(fwd) == 8 and len(grad) == 48, (sorted(fwd), sorted(grad))
    for n, k in {**fwd, **grad}.items():
        assert k[".vgpr_spill_count"] == 0, n
        # forward_kernel<PADW, ROWS, threads>: ROWS units hold their weights in
        # flight; grad_kernel<PADW, k, FORM, MANY>: bands of
        # small images
        few = re.search("14forward_kernelILb[01]ELb1E|11grad_kernelILb[01]ELi[2-7]ELi[12]E", n)
        assert waves(k) >= (3 if few else 4), (n, k[".vgpr_count"])
