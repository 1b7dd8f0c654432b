"""GPU parity of the one-pass X-cache kernel in each of its shapes (4, 6, 8 and 10 waves, 16 or 32 heads per group)
against the fp64 oracle, at widths that leave column owners without columns, head counts on either side of a group,
one row, a row on either side of a tile, and batches whose splits take more than one round of workgroups."""
import numpy as np
import pytest

from paper_2503_05840_amd import synth
from gpu_harness import TOL, XCase, say

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, d_model, d_k, T, lens)
    (1, 16, 512, 32, 33, None), (3, 17, 512, 32, 700, [700, 1, 32]), (2, 8, 640, 64, 31, None), (1, 40, 640, 32, 1, None),
    (5, 16, 768, 32, 65, [65, 64, 63, 1, 33]), (2, 33, 768, 32, 600, None), (1, 16, 896, 32, 520, None), (2, 9, 1024, 32, 90, [90, 5]),
    (9, 32, 1024, 32, 40, None), (24, 20, 1280, 32, 300, None), (70, 8, 512, 32, 300, None), (3, 16, 1152, 32, 97, [97, 96, 1]),
]


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_one_pass_xcache_shapes_match_oracle(i):
    B, H, d, d_k, T, lens = SHAPES[i]
    cfg = synth.scaled(synth.CONFIGS[4], B=B, H=H, d=d, d_k=d_k, T=T)
    say(f"[case] one-pass X-cache {i}: B={B} H={H} d_model={d} d_k={d_k} T={T} lens={lens}")
    x = XCase(cfg, q_scale=[1.0, 4.0][i % 2], lens=lens, oracle_seqs=None if B < 20 else {0, B - 1})
    a = x.run()
    e = x.err(a)
    say(f"  rel err {e:.3e}")
    assert e <= TOL["bf16"]
    assert np.array_equal(a, x.run())


@pytest.mark.parametrize("d_k", [96, 128, 160, 256])
def test_xcache_heads_on_either_side_of_128_columns_match_oracle(d_k):
    # 128 columns are the widest head of the MFMA path; wider ones take the plain kernels
    cfg = synth.scaled(synth.CONFIGS[4], B=2, H=3, d=512, d_k=d_k, T=70)
    say(f"[case] X-cache, heads of {d_k} columns: B=2 H=3 d_model=512 T=70")
    x = XCase(cfg, lens=[70, 33])
    e = x.err(x.run())
    say(f"  rel err {e:.3e}")
    assert e <= TOL["bf16"]
