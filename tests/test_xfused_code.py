"""What the compiler made of the one-pass X-cache kernel, of the wide path's weighted sum and of the stream kernel, read from the built library: no scratch memory in any
instantiation, and a partial that leaves by buffer stores, without a predicate and a 64-bit address for each piece."""
import re

import pytest

import built_code

XFUSED = "_ZN4slim12_GLOBAL__N_113xfused_kernelI"
KWEIGHTED = "_ZN4slim12_GLOBAL__N_116kweighted_kernelI"
STREAM = "_ZN4slim12_GLOBAL__N_119fused_stream_kernelI"


def _scratch(prefix, folder):
    """{kernel: bytes of scratch a lane}"""
    blocks = re.split(r"\n\s+- \.agpr_count", built_code.notes(prefix, folder))[1:]
    found = {re.search(r"\.name:\s+(\S+)", b).group(1): int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", b).group(1)) for b in blocks}
    return {name: size for name, size in found.items() if name.startswith(prefix)}


@pytest.mark.skipif(not built_code.PRESENT, reason="no disassembler")
@pytest.mark.parametrize("prefix,kernels", [(XFUSED, 12), (KWEIGHTED, 2), (STREAM, 32)])
def test_no_scratch(prefix, kernels, tmp_path):
    found = _scratch(prefix, tmp_path)
    assert len(found) >= kernels and not any(found.values()), found


@pytest.mark.skipif(not built_code.PRESENT, reason="no disassembler")
def test_partials_leave_by_buffer_stores(tmp_path):
    for name in _scratch(XFUSED, tmp_path):
        blocks, half, tiles = (int(x) for x in re.match(r"Li(\d)ELi(\d)ELi(\d)E", name[len(XFUSED):]).groups())
        text = built_code.disassembly(name, tmp_path)
        assert text.count("buffer_store_dwordx4") % (tiles * (8 * blocks + 4 * half)) == 0 and "buffer_store_dwordx4" in text, name
        assert "global_store_dwordx4" not in text, name
