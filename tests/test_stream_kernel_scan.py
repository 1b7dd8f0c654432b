"""The kernels that add up the sequences' tiles do it in registers, looked for in the built library's code: no step of the scan over the lanes goes
through LDS.  By shuffles it cost each launch 0.2 to 0.4 us."""
import pytest

import built_code

STREAM = "_ZN4slim12_GLOBAL__N_119fused_stream_kernelILi%dELb%dELi%dELb%dEEEvNS_9FusedArgsE"
PROJECT = "_ZN4slim12_GLOBAL__N_119project_mfma_kernelILi%dELb0ELb0ELb%dEEEvNS_8ProjArgsE"


@pytest.mark.skipif(not built_code.PRESENT, reason="no disassembler")
@pytest.mark.parametrize("name", [STREAM % k for k in ((1, 0, 8, 0), (1, 0, 8, 1), (1, 1, 16, 1), (2, 0, 16, 0), (2, 1, 16, 0), (2, 0, 16, 1))] +
                         [PROJECT % k for k in ((1, 0), (1, 1), (4, 0))])
def test_tiles_are_added_up_in_registers(name, tmp_path):
    text = built_code.disassembly(name, tmp_path)
    assert "v_mfma" in text and "row_bcast" in text
    assert "ds_bpermute" not in text
