"""The gfx950 code objects inside the built library: what its kernels reserve
(their kernel descriptors) and, through llvm-objdump, their instructions."""
import os
import re
import struct
import subprocess

import paper_2603_19610_amd as pv

LLVM = "/opt/rocm/llvm/bin"
_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _sections(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, num, strx = struct.unpack_from("<HHH", elf, 0x3A)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * size) for i in range(num)]
    names = elf[heads[strx][4]:heads[strx][4] + heads[strx][5]]
    return [(names[h[0]:names.index(b"\0", h[0])].decode(), h) for h in heads]


def code_objects(path=pv.LIB_PATH):
    """The gfx950 ELF images of the library, one per source file."""
    data = open(path, "rb").read()
    out = []
    for name, h in _sections(data):
        if name != ".hip_fatbin":
            continue
        fat = data[h[4]:h[4] + h[5]]
        for m in re.finditer(re.escape(_MAGIC), fat):
            n, = struct.unpack_from("<Q", fat, m.start() + len(_MAGIC))
            at = m.start() + len(_MAGIC) + 8
            for _ in range(n):
                off, size, idlen = struct.unpack_from("<QQQ", fat, at)
                target = fat[at + 24:at + 24 + idlen].decode()
                at += 24 + idlen
                if "gfx950" in target and size:
                    out.append(fat[m.start() + off:m.start() + off + size])
    assert out, f"no gfx950 code object in {path}"
    return out


def kernels():
    """{mangled name: (registers a wave reserves, fixed LDS bytes)}."""
    res = {}
    for elf in code_objects():
        sec = _sections(elf)
        tab = next(h for name, h in sec if name == ".symtab" or name == ".dynsym")
        strs = sec[tab[6]][1]
        for at in range(tab[4], tab[4] + tab[5], 24):
            name, _, _, shndx, value, size = struct.unpack_from("<IBBHQQ", elf, at)
            s = elf[strs[4] + name:elf.index(b"\0", strs[4] + name)].decode()
            if not s.endswith(".kd"):
                continue
            h = sec[shndx][1]
            kd = elf[h[4] + value - h[3]:][:64]
            lds, = struct.unpack_from("<I", kd, 0)
            rsrc1, = struct.unpack_from("<I", kd, 48)
            res[s[:-3]] = (((rsrc1 & 63) + 1) * 8, lds)  # granules of 8 registers
    return res


def disassembly(tmp_path):
    """Lists of instructions (text) of every code object, in order."""
    out = []
    for i, elf in enumerate(code_objects()):
        p = os.path.join(tmp_path, f"obj{i}.elf")
        open(p, "wb").write(elf)
        r = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", p],
                           capture_output=True, text=True, check=True)
        lines = (l.split("//")[0].strip() for l in r.stdout.splitlines())
        out.append([l for l in lines if l])
    return out
