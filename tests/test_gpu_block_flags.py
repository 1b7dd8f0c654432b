"""The first launch of an attention block hands its row splits over by flags that nothing has cleared: any contents of the
workspace (zeros, all ones, what another shape's call left) give the same bits.  Two row splits to eight, one unit to the most
that are split (96 for the slim block's two matrices at 33 sequences; the vanilla block's 144 there are not)."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import BlockCase, TOL, row_rel_err, say

pytestmark = pytest.mark.gpu

SHAPES = [(1, 4, 128, 40, None), (3, 16, 128, 60, 10000.0), (33, 16, 64, 20, None), (17, 8, 96, 33, 10000.0)]   # (B, H, d_k, T, rope)


@pytest.mark.parametrize("i", range(len(SHAPES)))
def test_block_takes_any_workspace(i):
    import torch
    B, H, d_k, T, rope = SHAPES[i]
    say(f"[case] block, workspace contents: B={B} H={H} d_k={d_k} T={T} rope={rope}")
    k = BlockCase(synth.scaled(synth.CONFIGS[1], B=B, H=H, d=H * d_k, d_k=d_k, T=T, len_lo=2), rope_base=rope)
    ws = torch.zeros(binding.slim_workspace_bytes_block(B, H, T, H * d_k, "bf16"), dtype=torch.uint8, device="cuda")
    first = k.run_slim(workspace=ws)
    vfirst = k.run_vanilla(workspace=ws)
    assert row_rel_err(first[0], k.ref) <= TOL["bf16"] and row_rel_err(first[1], k.k_new) <= TOL["bf16"]
    assert row_rel_err(vfirst[0], k.ref) <= TOL["bf16"]
    for fill in (255, 0, 1):
        ws.fill_(fill)
        for _ in range(2):
            for a, b in zip(first + vfirst, k.run_slim(workspace=ws) + k.run_vanilla(workspace=ws)):
                assert np.array_equal(a, b)
