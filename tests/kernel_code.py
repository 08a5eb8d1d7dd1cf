"""The gfx950 code objects inside the built library: each kernel's resources (from the code object's metadata) and its instructions."""
import functools
import os
import struct
import subprocess
import tempfile

import msgpack

from paper_2411_01075_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def _code_objects(data):
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in target and size:
                yield data[at + offset:at + offset + size]
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _kernels(elf):
    """The kernel entries of the code object's metadata note (a msgpack map, note type 32)."""
    section, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        _, kind, _, _, offset, size = struct.unpack_from("<IIQQQQ", elf, section + k * entry)
        q, end = offset, offset + size
        while kind == 7 and q < end:
            name, desc, note = struct.unpack_from("<III", elf, q)
            d = q + 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[d:d + desc], strict_map_key=False)["amdhsa.kernels"]
            q = d + (desc + 3) // 4 * 4


@functools.lru_cache(maxsize=None)
def _all():
    if not os.path.exists(build.LIB):
        build.build(verbose=False)
    with open(build.LIB, "rb") as f:
        data = f.read()
    return {k[".name"]: (k, elf) for elf in _code_objects(data) for k in _kernels(elf)}


def kernels(part):
    """{mangled name: metadata} of the kernels whose mangled name contains `part`."""
    found = {n: k for n, (k, _) in _all().items() if part in n}
    assert found, part
    return found


def instructions(name):
    """The kernel's instructions, one text each."""
    with tempfile.NamedTemporaryFile(suffix=".co") as f:
        f.write(_all()[name][1])
        f.flush()
        out = subprocess.run([OBJDUMP, "--disassemble-symbols=" + name, "--no-show-raw-insn", f.name], check=True, capture_output=True, text=True).stdout
    return [line.split("//")[0].strip() for line in out.splitlines() if line.startswith("\t")]
