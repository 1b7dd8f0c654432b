"""The tile prefix on either side of the lane rows (16), of the wave (64) and of two waves' worth of sequences, ragged with sequences of one tile and of
several, in the single launch, by context and by sequence: every sequence against the fp64 oracle, at the tolerance of bf16 caches."""
import numpy as np
import pytest

from paper_2503_05840_amd import synth
from gpu_harness import TOL, KCase, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H", [(B, 4) for B in (2, 15, 16, 17, 32, 33, 63, 64, 65, 128, 129, 150)] + [(64, 20), (65, 20), (150, 20)])
def test_sequences_on_either_side_of_a_wave_match_oracle(B, H):
    cfg = synth.scaled(synth.CONFIGS[3], B=B, H=H, d=H * 64, T=130)
    for lens in ([1 + (53 * b + 7 * H) % 130 for b in range(B)], [130] * B):
        say(f"[case] tile prefix: B={B} H={H} lens={lens[:3]}..")
        k = KCase(cfg, lens=lens, need_v=False)
        a = k.run_slim()
        e = k.err(a)
        say(f"  rel err {e:.3e}")
        assert e <= TOL["bf16"]
        assert np.array_equal(a, k.run_slim())
