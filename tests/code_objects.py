"""What the compiler noted about the kernels of the built library: the metadata of the gfx950 code
objects inside libpowergossip.so (register counts, arguments).  No GPU and no tool is needed."""
import struct
import subprocess

import msgpack


def _notes(elf):
    """Descriptors of the AMDGPU metadata notes (type 32) of one ELF64 image."""
    shoff = struct.unpack_from("<Q", elf, 0x28)[0]
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + k * size + 4)
        off, length = struct.unpack_from("<QQ", elf, shoff + k * size + 0x18)
        if kind != 7:                                  # SHT_NOTE
            continue
        at = off
        while at < off + length:
            nlen, dlen, typ = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (nlen + 3) // 4 * 4
            if typ == 32:
                yield elf[desc:desc + dlen]
            at = desc + (dlen + 3) // 4 * 4


def kernels(library):
    """{demangled name without arguments: metadata} of every kernel in the library."""
    blob = open(library, "rb").read()
    magic, found, at = b"__CLANG_OFFLOAD_BUNDLE__", [], 0
    while (at := blob.find(magic, at)) >= 0:
        pos = at + len(magic)
        n, = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, pos)
            triple = blob[pos + 24:pos + 24 + tlen]
            pos += 24 + tlen
            if b"gfx950" in triple and size:
                for desc in _notes(blob[at + off:at + off + size]):
                    found += msgpack.unpackb(desc, strict_map_key=False)["amdhsa.kernels"]
        at += len(magic)
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True,
                           text=True, check=True).stdout.split("\n")
    return {name.split("(")[0].replace("void ", ""): k for name, k in zip(names, found)}


def arguments(kernel):
    """Arguments a launch passes (the hidden ones the runtime fills in left out)."""
    return sum(not a[".value_kind"].startswith("hidden") for a in kernel[".args"])
