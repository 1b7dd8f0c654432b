"""The merge of a projection's partials on either side of the four sequences up to which they are fetched four at a time, with one, two,
three, four, five and more partials a sequence, and with fewer rows than splits: against the fp64 oracle, at the tolerance of bf16 caches."""
import numpy as np
import pytest

from paper_2503_05840_amd import synth
from gpu_harness import TOL, XCase, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 3, 4, 5, 20])
@pytest.mark.parametrize("T", [40, 200, 330, 500, 600, 1200])
def test_partials_of_few_sequences_match_oracle(B, T):
    # (one head group: a split per 128 rows; 20 sequences: a batch chunk of sixteen and one of four)
    lens = [max(1, T - 97 * b % T) for b in range(B)]
    cfg = synth.scaled(synth.CONFIGS[4], B=B, H=6, d=512, d_k=32, T=T)
    say(f"[case] partials of few sequences: B={B} T={T}")
    x = XCase(cfg, lens=lens)
    a = x.run()
    e = x.err(a)
    say(f"  rel err {e:.3e}")
    assert e <= TOL["bf16"]
    assert np.array_equal(a, x.run())
