"""The gfx950 code objects inside a built library: their kernels' metadata and their disassembly."""
import os
import re
import struct
import subprocess

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def code_objects(path):
    """The ELF files of the library's offload bundles."""
    data = open(path, "rb").read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        entry = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", data, entry - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, entry)
            entry += 24 + n
            elf = data[at + off:at + off + size]
            if elf[:4] == b"\x7fELF":
                yield elf
        at += len(magic)


def kernel_metadata(path):
    """{kernel symbol: metadata}: the AMDGPU note (type 32) holds the compiler's record of each kernel as MessagePack."""
    import msgpack
    out = {}
    for elf in code_objects(path):
        shoff = struct.unpack_from("<Q", elf, 40)[0]
        shentsize, shnum = struct.unpack_from("<HH", elf, 58)
        for i in range(shnum):
            typ, _, _, start, length = struct.unpack_from("<IQQQQ", elf, shoff + i * shentsize + 4)
            if typ != 7:                                      # SHT_NOTE
                continue
            p = start
            while p < start + length:
                namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
                desc = p + 12 + (namesz + 3) // 4 * 4
                if ntype == 32:
                    for k in msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]:
                        out[k[".name"]] = k
                p = desc + (descsz + 3) // 4 * 4
    return out


def disassembly(path, tmp):
    """{function symbol: [(address, instruction text)]}"""
    out = {}
    for i, elf in enumerate(code_objects(path)):
        name = os.path.join(tmp, f"{i}.elf")
        with open(name, "wb") as f:
            f.write(elf)
        text = subprocess.run([OBJDUMP, "-d", name], check=True, capture_output=True, text=True).stdout
        body = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if m:
                body = out.setdefault(m.group(1), [])
                continue
            m = re.match(r"\s+(\S.*?)\s*// ([0-9A-F]+):", line)
            if m and body is not None:
                body.append((int(m.group(2), 16), m.group(1)))
    return out
