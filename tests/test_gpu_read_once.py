"""GPU parity of the block's products where their loads of W are nontemporal: four matrices of together at least 96 MB, each
read by one batch chunk.  One sequence, and 17: a second batch tile with one sequence, rows of W split over workgroups."""
import numpy as np
import pytest

from paper_2503_05840_amd import synth
from gpu_harness import BlockCase, TOL, row_rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 17])
def test_products_of_large_matrices(B):
    say(f"[case] products of large matrices B={B}")
    cfg = synth.scaled(synth.CONFIGS[1], B=B, H=28, d=3584, d_k=128, T=20, len_lo=3)
    assert 4 * 2 * cfg.d ** 2 >= 96 << 20
    k = BlockCase(cfg)
    y, krow = k.run_slim()
    assert row_rel_err(y, k.ref) <= TOL["bf16"] and row_rel_err(krow, k.k_new) <= TOL["bf16"]
    assert np.array_equal(y, k.run_slim()[0])
    y, krow, vrow = k.run_vanilla()
    assert row_rel_err(y, k.ref) <= TOL["bf16"] and row_rel_err(krow, k.k_new) <= TOL["bf16"] and row_rel_err(vrow, k.v_new) <= TOL["bf16"]
