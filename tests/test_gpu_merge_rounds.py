"""GPU parity of the fp32 merge + projection around its rounds of 16 splits (one split per 32 rows here): either side of 16, 32,
48 and at the most, 64; rows that are no whole 64-row chunk; a ragged batch whose shorter sequences lack splits, whose place in
the scratch holds NaN."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import KCase, TOL, say

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, d_k, T, len_lo)
    (1, 1, 16, 512, 0), (2, 3, 16, 513, 40), (3, 2, 32, 1024, 1), (5, 5, 16, 1025, 33), (4, 2, 80, 1536, 31), (1, 17, 16, 1537, 0), (3, 4, 64, 2048, 5),
    (2, 1, 48, 3000, 64),
]


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_merge_of_many_splits(i):
    import torch
    B, H, d_k, T, lo = SHAPES[i]
    cfg = synth.scaled(synth.CONFIGS[0], B=B, H=H, d=H * d_k, d_k=d_k, T=T, len_lo=lo)
    say(f"[case] merge of many splits {i}: B={B} H={H} d_k={d_k} T={T} len_lo={lo}")
    k = KCase(cfg, q_scale=8.0, need_v=False)
    ws = torch.full((binding.slim_workspace_bytes(B, H, T, H * d_k, "f32") // 4,), float("nan"), device="cuda").view(torch.uint8)
    a = k.run_slim(workspace=ws)
    e = k.err(a)
    say(f"  rel err {e:.3e}")
    assert e <= TOL["f32"]
    assert np.array_equal(a, k.run_slim(workspace=ws))
