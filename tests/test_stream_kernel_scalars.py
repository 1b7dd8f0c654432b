"""Scalars that the single launch keeps in lanes of vector registers, counted in the built library's code: the order of its
arguments decides how many there are, and with ~390 (or 360) small layers took 2 us of 20 longer than with ~300 (or 270)."""
import os
import struct
import subprocess

import pytest

from paper_2503_05840_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
KERNEL = "_ZN4slim12_GLOBAL__N_119fused_stream_kernelILi1ELb0ELi%dELb0EEEvNS_9FusedArgsE"


def _code_objects(blob):
    """The gfx950 code objects of a library: bundles of {entries, then offset, size, length of the name, name per entry}."""
    at = blob.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        n, pos = struct.unpack_from("<Q", blob, pos)[0], pos + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, pos)
            pos += 24
            name = blob[pos:pos + length]
            pos += length
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, pos)


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no disassembler")
@pytest.mark.parametrize("columns,most", [(8, 300), (16, 275)])
def test_single_launch_of_few_heads(columns, most, tmp_path):
    if not os.path.exists(build.LIB):
        build.build()
    symbol = KERNEL % columns
    with open(build.LIB, "rb") as f:
        objects = [o for o in _code_objects(f.read()) if symbol.encode() in o]
    assert len(objects) == 1
    path = tmp_path / "code.o"
    path.write_bytes(objects[0])
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--disassemble-symbols=" + symbol, str(path)], check=True, capture_output=True, text=True).stdout
    assert text.count("v_mfma") > 0
    assert text.count("v_readlane_b32") <= most
