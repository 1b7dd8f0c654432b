"""GPU parity of the wide K-cache path's numerators per 64-row block: sizes at the edges of 64-row blocks, 32-row tiles and
16-row waves, splits of whole blocks with empty ones, scores peaky enough that the blocks' references differ by tens of
powers of two, every lane count per head, and (the last two) shapes whose scratch has no room for the blocks' references,
which take the scores instead.  Tolerances as in test_gpu_wide.py: the oracle's, and 5e-5 against the plain fp32 kernels
(both weigh in fp32; what differs is the projection's split of C into two bf16 terms, 2^-17 per term)."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import KCase, TOL, head_rel_err, say

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, d_k, T, len_lo, rope base, query scale)
    (1, 34, 64, 65, 0, None, 8.0), (2, 40, 32, 127, 30, None, 30.0), (3, 48, 16, 128, 1, None, 30.0), (1, 40, 128, 577, 0, None, 30.0),
    (5, 64, 32, 449, 3, 10000.0, 30.0), (2, 33, 128, 1100, 60, 10000.0, 8.0), (2, 48, 8, 400, 20, None, 8.0), (1, 64, 8, 1000, 0, None, 8.0),
]


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_wide_kcache_blocks(i):
    B, H, d_k, T, lo, rope, q_scale = SHAPES[i]
    d = H * d_k
    assert d % 128 == 0
    cfg = synth.scaled(synth.CONFIGS[1], B=B, H=H, d=d, d_k=d_k, T=T, len_lo=lo)
    say(f"[case] wide K-cache blocks {i}: B={B} H={H} d_k={d_k} T={T} len_lo={lo} rope={rope} q x{q_scale}")
    k = KCase(cfg, q_scale=q_scale, rope_base=rope, need_v=False)
    a, g = k.run_slim(), k.run_slim(variant=binding.VARIANT_GENERIC)
    e, dd = k.err(a), head_rel_err(a, g.astype(np.float64), H)
    say(f"  rel err {e:.3e}, against the plain kernels {dd:.3e}")
    assert e <= TOL["bf16"] and dd <= 5e-5
    assert np.array_equal(a, k.run_slim())
