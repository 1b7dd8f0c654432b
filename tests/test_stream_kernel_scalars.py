"""Scalars that the single launch keeps in lanes of vector registers, counted in the built library's code: the order of its
arguments decides how many there are, and with ~390 (or 360) small layers took 2 us of 20 longer than with ~300 (or 270)."""
import pytest

import built_code

KERNEL = "_ZN4slim12_GLOBAL__N_119fused_stream_kernelILi1ELb0ELi%dELb0EEEvNS_9FusedArgsE"


@pytest.mark.skipif(not built_code.PRESENT, reason="no disassembler")
@pytest.mark.parametrize("columns,most", [(8, 300), (16, 275)])
def test_single_launch_of_few_heads(columns, most, tmp_path):
    text = built_code.disassembly(KERNEL % columns, tmp_path)
    assert text.count("v_mfma") > 0
    assert text.count("v_readlane_b32") <= most
