"""GPU parity of the stream kernel at the share length from which its first four waves take a tile more (32 tiles of a group's
range): shares of 31, 32 and 33 tiles, a last group that is shorter, a last tile of one row, and ragged sequences whose ends
leave shares on either side of it, plain and rotary keys, one and two head tiles, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import KCase, TOL, say

pytestmark = pytest.mark.gpu

CASES = [  # (H, d_k, T, lens, rope base): 17 heads of 72 columns are 8 groups, 16 heads 16 groups
    (17, 72, 31 * 8 * 32, None, None), (17, 72, 31 * 8 * 32 + 1, None, None), (17, 72, 32 * 8 * 32 - 32, None, 10000.0),
    (17, 72, 32 * 8 * 32, None, None), (17, 72, 32 * 8 * 32 + 1, None, 10000.0), (17, 72, 33 * 8 * 32, None, None),
    (16, 72, 32 * 16 * 32 - 31, None, None), (17, 72, 4000, [4000, 3000, 1025, 300], None), (17, 72, 6000, [993, 6000, 1700, 31], 10000.0),
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_shares_around_the_lead_match_oracle(i):
    H, d_k, T, lens, rope = CASES[i]
    B = len(lens) if lens else 1
    say(f"[case] tile lead {i}: B={B} H={H} d_k={d_k} T={T} lens={lens} rope={rope}")
    k = KCase(synth.scaled(synth.CONFIGS[1], B=B, H=H, d=H * d_k, d_k=d_k, T=T), q_scale=8.0, lens=lens, rope_base=rope, need_v=False)
    assert binding.auto_variant_name(B, H, T, H * d_k, "bf16") == "fused"
    a = k.run_slim()
    e = k.err(a)
    say(f"  rel err {e:.3e}")
    assert e <= TOL["bf16"]
    assert np.array_equal(a, k.run_slim())
