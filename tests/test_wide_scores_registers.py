"""The score kernel of wide K-caches with rotary keys has its 16 rows of K and the table's entries of four of them in flight together:
64 and 32 registers, counted in the built library.  With 64 in all it loaded a few rows at a time (12.6 instead of 8.1 us at 2 x 3000 x 40 x 64)."""
import pytest

import built_code

KERNEL = "_ZN4slim12_GLOBAL__N_114kscores_kernelILi%dELb1ELb1EEEvPKfPKtlPKiiiiifS3_PfS8_Pii"


@pytest.mark.skipif(not built_code.PRESENT, reason="no disassembler")
@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16])
def test_rotary_scores_keep_their_rows_in_flight(lanes, tmp_path):
    assert built_code.vector_registers(KERNEL % lanes, tmp_path) >= 16 * 4 + 4 * 8
