"""What the compiler made of the one-pass X-cache kernel, of the wide path's weighted sum and of the stream kernel, read from the built library: no scratch memory in any
instantiation."""
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
