"""The gfx950 code in the built library, kernel by kernel.  Not a test module."""
import os
import re
import struct
import subprocess

from paper_2503_05840_amd import build

LLVM = "/opt/rocm/llvm/bin/"
PRESENT = all(os.path.exists(LLVM + tool) for tool in ("llvm-objdump", "llvm-readelf"))
_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """Bundles of {number of entries, then offset, size, length of the name, name of each}."""
    at = blob.find(_MAGIC)
    while at >= 0:
        pos = at + len(_MAGIC)
        n, pos = struct.unpack_from("<Q", blob, pos)[0], pos + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, pos)
            pos += 24
            name = blob[pos:pos + length]
            pos += length
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(_MAGIC, pos)


def _file_with(symbol, folder):
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        found = [o for o in _code_objects(f.read()) if symbol.encode() in o]
    assert len(found) == 1, symbol
    path = os.path.join(str(folder), "code.o")
    with open(path, "wb") as f:
        f.write(found[0])
    return path


def _output(*cmd):
    return subprocess.run(cmd, check=True, capture_output=True, text=True).stdout


def disassembly(symbol, folder):
    return _output(LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", "--disassemble-symbols=" + symbol, _file_with(symbol, folder))


def notes(symbol, folder):
    return _output(LLVM + "llvm-readelf", "--notes", _file_with(symbol, folder))


def vector_registers(symbol, folder):
    return int(re.search(r"\.name:\s+%s\n(?:(?!\s*\.name:).*\n)*?.*\.vgpr_count:\s+(\d+)" % re.escape(symbol), notes(symbol, folder)).group(1))
