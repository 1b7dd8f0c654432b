"""The one-pass X-cache kernel where its steps differ: one, two, three and four tiles of rows a workgroup (the first, the middle and the
last of its loop), with every block shape of a wave's columns, and queries large enough that references move between tiles.
Tolerance: the one of bf16 caches; with moving references against an oracle that sees the weights as stored, because scores this large turn
the rounding of W_K into more than the tolerance."""
import numpy as np
import pytest

from paper_2503_05840_amd import synth
from gpu_harness import TOL, XCase, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [16, 20])
@pytest.mark.parametrize("d", [512, 640, 768, 896, 1024, 1152, 1280])
def test_steps_of_the_one_pass_kernel_match_oracle(d, H):
    # (300 sequences of up to 127 rows: one split each, so that a workgroup goes through all tiles of a sequence)
    lens = [1 + (37 * b + 11 * d) % 127 for b in range(300)]
    lens[:6] = [127, 96, 64, 32, 33, 97]
    cfg = synth.scaled(synth.CONFIGS[4], B=300, H=H, d=d, d_k=32, T=127)
    for q_scale in (1.0, 60.0):
        say(f"[case] steps of the one-pass X-cache: H={H} d_model={d} q x {q_scale}")
        x = XCase(cfg, q_scale=q_scale, lens=lens, oracle_seqs=set(range(0, 300, 60)) | set(range(6)), oracle_sees_rounded_weights=q_scale > 1.0)
        a = x.run()
        e = x.err(a)
        say(f"  rel err {e:.3e}")
        assert e <= TOL["bf16"]
        assert np.array_equal(a, x.run())
