"""The first launch of an attention block hands its row splits over by flags that nothing has cleared: any contents of the
workspace (zeros, all ones, what blocks of another shape left) give the same bits.  Two row splits to eight; of the slim block's
two matrices 6 units, the fewest that are split, to 128, the most, whose 256 flags are all there are (the vanilla block's 144 or
192 units at 17 and 33 sequences are not split)."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import BlockCase, TOL, row_rel_err, say
from launch_rules import batch_chunks, row_splits

pytestmark = pytest.mark.gpu

SHAPES = [  # (B, H, d_k, T, rope)
    (1, 4, 128, 40, None), (3, 16, 128, 60, 10000.0), (33, 16, 64, 20, None), (17, 8, 96, 33, 10000.0),
    (17, 32, 16, 40, None), (2, 3, 128, 50, 10000.0),
]


def _units_and_splits(i, matrices):
    B, H, d_k = SHAPES[i][:3]
    d, n = H * d_k, H * matrices
    return n * batch_chunks(B, d, d, n), row_splits(n, d, d, B)


def test_shapes_reach_the_ends_of_the_range():
    got = [_units_and_splits(i, 2) for i in range(len(SHAPES))]
    assert min(got)[0] == 6 and max(got) == (128, 2)              # 128 units x 2: the last of 256 flags
    assert min(c for _, c in got) == 2 and max(c for _, c in got) == 8
    assert [_units_and_splits(i, 3) for i in (2, 4)] == [(144, 1), (192, 1)]


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_block_takes_any_workspace(i):
    import torch
    B, H, d_k, T, rope = SHAPES[i]
    say(f"[case] block, workspace contents: B={B} H={H} d_k={d_k} T={T} rope={rope}")
    k = BlockCase(synth.scaled(synth.CONFIGS[1], B=B, H=H, d=H * d_k, d_k=d_k, T=T, len_lo=2), rope_base=rope)
    # a block of another shape, with other units and splits, for the same workspace
    oB, oH, od_k, oT, orope = SHAPES[(i + 1) % len(SHAPES)]
    other = BlockCase(synth.scaled(synth.CONFIGS[1], B=oB, H=oH, d=oH * od_k, d_k=od_k, T=oT, len_lo=2), rope_base=orope)
    size = max(binding.slim_workspace_bytes_block(B, H, T, H * d_k, "bf16"), binding.slim_workspace_bytes_block(oB, oH, oT, oH * od_k, "bf16"))
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    first = k.run_slim(workspace=ws)
    vfirst = k.run_vanilla(workspace=ws)
    assert row_rel_err(first[0], k.ref) <= TOL["bf16"] and row_rel_err(first[1], k.k_new) <= TOL["bf16"]
    assert row_rel_err(vfirst[0], k.ref) <= TOL["bf16"]
    for fill in (255, 0, 1, None):
        if fill is None:
            other.run_slim(workspace=ws)
            other.run_vanilla(workspace=ws)
        else:
            ws.fill_(fill)
        for _ in range(2):
            for a, b in zip(first + vfirst, k.run_slim(workspace=ws) + k.run_vanilla(workspace=ws)):
                assert np.array_equal(a, b)
