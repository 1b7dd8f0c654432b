"""GPU parity at head widths whose column groups of 8 are no whole fours (their partial sums are padded on the way from the
workgroups that share the rows of W to the last of them): the single launch, a projection of its own with one and with two
batch tiles, and the dense products of a block, few elements (columns in order) and many, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import BlockCase, KCase, TOL, row_rel_err, say

pytestmark = pytest.mark.gpu
BASE = synth.CONFIGS[1]


@pytest.mark.parametrize("d_k", [16, 24, 40, 48, 56, 72, 80, 88, 104, 112, 120])
def test_head_widths_match_oracle(d_k):
    H = 7 if d_k >= 72 else 19                           # (rows of W for two to four workgroups)
    for B, T in ((1, 33), (3, 150), (20, 64), (70, 40)):
        say(f"[case] head width {d_k}: B={B} H={H} T={T}")
        k = KCase(synth.scaled(BASE, B=B, H=H, d=H * d_k, d_k=d_k, T=T, len_lo=1), q_scale=4.0, need_v=False)
        a = k.run_slim()
        e = k.err(a)
        say(f"  rel err {e:.3e}")
        assert e <= TOL["bf16"]
        assert np.array_equal(a, k.run_slim(variant=binding.VARIANT_VIA_MEMORY))


# (a workgroup's B x d_k elements: up to 512 and up to 1024 in column order, one and two a thread, more in the padded order)
@pytest.mark.parametrize("d_k", [16, 48, 64, 80, 112])
@pytest.mark.parametrize("B", [2, 8, 9, 16])
def test_blocks_of_these_widths_match_oracle(d_k, B):
    H = 7 if d_k >= 72 else 19
    say(f"[case] block, head width {d_k}: B={B} H={H} T=50")
    b = BlockCase(synth.scaled(BASE, B=B, H=H, d=H * d_k, d_k=d_k, T=50, len_lo=1), rope_base=10000.0)
    y, krow = b.run_slim()
    yv, _, _ = b.run_vanilla()
    say(f"  rel err {row_rel_err(y, b.ref):.3e}, vanilla {row_rel_err(yv, b.ref):.3e}")
    assert row_rel_err(y, b.ref) <= TOL["bf16"] and row_rel_err(yv, b.ref) <= TOL["bf16"]
    assert row_rel_err(krow, b.k_new) <= TOL["bf16"]
