"""GPU parity of the fp32 stream kernel and the vector-ALU merge + projection against the fp64 oracle, at the
sizes where they can go wrong: one row, a row on either side of a 32-row tile, rows that are no multiple of the
64-column blocks or of a wave's 256-column pieces, both head tiles with padded heads, more tiles than splits,
a head wider than one 64-column block of the projection, more sequences than its chunk of four."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import KCase, TOL, say

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, d_k, T, len_lo, rope base, query scale)
    (1, 1, 16, 1, 0, None, 1.0), (2, 3, 16, 31, 0, 10000.0, 8.0), (1, 8, 64, 32, 0, None, 8.0), (3, 5, 48, 33, 1, 10000.0, 30.0),
    (1, 16, 64, 65, 0, None, 50.0), (5, 17, 16, 130, 1, None, 8.0), (2, 12, 64, 700, 90, 500.0, 30.0), (1, 32, 32, 2200, 0, None, 8.0),
    (1, 2, 400, 300, 0, None, 8.0), (7, 1, 1024, 45, 20, None, 1.0), (70, 4, 32, 40, 1, 10000.0, 8.0), (300, 2, 16, 9, 1, None, 2000.0),
]


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_f32_stream_matches_oracle(i):
    B, H, d_k, T, lo, rope, q_scale = SHAPES[i]
    cfg = synth.scaled(synth.CONFIGS[0], B=B, H=H, d=H * d_k, d_k=d_k, T=T, len_lo=lo)
    say(f"[case] f32 stream {i}: B={B} H={H} d_k={d_k} T={T} len_lo={lo} rope={rope} q x{q_scale}")
    k = KCase(cfg, q_scale=q_scale, rope_base=rope, need_v=False)
    a = k.run_slim()
    e, eg = k.err(a), k.err(k.run_slim(variant=binding.VARIANT_GENERIC))
    say(f"  rel err {e:.3e}, plain kernels {eg:.3e}")
    assert e <= TOL["f32"] and eg <= TOL["f32"]
    assert np.array_equal(a, k.run_slim())
