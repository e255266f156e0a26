"""The device code of the built libbitcos.so: each kernel's resource counts (from
the code objects' metadata notes) and its disassembly."""

import functools
import re
import struct
import subprocess
import tempfile

import msgpack

from paper_2609_16338_amd import build_lib

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


@functools.lru_cache(maxsize=1)
def code_objects():
    """The gfx950 ELF images of the library, one per source file with kernels."""
    with open(build_lib.LIB, "rb") as f:
        lib = f.read()
    out = []
    at = lib.find(BUNDLE)
    while at >= 0:
        p = at + len(BUNDLE)
        entries, = struct.unpack_from("<Q", lib, p)
        p += 8
        if entries < 16:  # the marker is also a string of the loader
            for _ in range(entries):
                off, size, named = struct.unpack_from("<QQQ", lib, p)
                target = lib[p + 24:p + 24 + named]
                p += 24 + named
                if build_lib.ARCH.encode() in target and size:
                    out.append(lib[at + off:at + off + size])
        at = lib.find(BUNDLE, at + len(BUNDLE))
    return out


def _notes(elf):
    """The amdhsa metadata map of one image."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        off, = struct.unpack_from("<Q", elf, shoff + i * shentsize + 24)
        if kind == 7:  # SHT_NOTE: name size, description size, type, name, description
            nsz, dsz, ntype = struct.unpack_from("<III", elf, off)
            if ntype == 32:  # NT_AMDGPU_METADATA
                start = off + 12 + (nsz + 3) // 4 * 4
                return msgpack.unpackb(elf[start:start + dsz])
    return {"amdhsa.kernels": []}


def _short(mangled):
    """Readable names ("bitcos_k::bitcos_fast_kernel<5, 32, true, true, false>") of mangled ones."""
    p = subprocess.run(["c++filt"], input="\n".join(mangled), stdout=subprocess.PIPE, text=True, check=True)
    return [l.replace("(anonymous namespace)", "anon").split("(")[0].removeprefix("void ") for l in p.stdout.splitlines()]


@functools.lru_cache(maxsize=1)
def kernels():
    """{kernel name: its metadata} of the whole library."""
    ks = [k for elf in code_objects() for k in _notes(elf)["amdhsa.kernels"]]
    return dict(zip(_short([k[".name"] for k in ks]), ks))


def disassembly(pattern):
    """{kernel name: its instructions} of the images with a kernel whose name matches."""
    out = {}
    for elf in code_objects():
        names = [k[".name"] for k in _notes(elf)["amdhsa.kernels"]]
        if not any(re.search(pattern, s) for s in (_short(names) if names else [])):
            continue
        with tempfile.NamedTemporaryFile() as f:
            f.write(elf)
            f.flush()
            p = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", f.name],
                               stdout=subprocess.PIPE, text=True, check=True)
        bodies, cur = {}, None
        for line in p.stdout.splitlines():
            m = re.match(r"^(?:[0-9a-f]+ )?<(\w+)>:$", line.strip())
            if m:
                cur = bodies.setdefault(m.group(1), []) if m.group(1) in names else cur
            elif cur is not None and line.strip():
                cur.append(line.split("//")[0].strip())
        for name, short in zip(bodies, _short(list(bodies))):
            if re.search(pattern, short):
                out[short] = bodies[name]
    return out
