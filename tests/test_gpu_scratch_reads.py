"""What an fp32 step reads of its workspace follows the rows in use, not the capacity: with contexts of 50 rows in a capacity of
2048 the partials of up to 64 splits per sequence have a place in the workspace (33 MB here) and two of them exist.  A loop over 16
workspaces, which the 256 MB memory-side cache does not hold, then takes as long as a loop on one of them.  Measured: 23.60 us
and 23.64; 25.11 and 28.16 (1.12 times as long) when the places of the other splits were read.  The bound lies half way."""
import statistics

import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import KCase, TOL, say

pytestmark = pytest.mark.gpu


def test_short_contexts_in_a_large_capacity():
    import torch
    B, H, d_k, T = 4, 32, 32, 2048
    lens = [50, 37, 50, 44]
    say("[case] reads of the workspace: 4 sequences of up to 50 rows, capacity 2048")
    k = KCase(synth.scaled(synth.CONFIGS[0], B=B, H=H, d=H * d_k, d_k=d_k, T=T, len_lo=0), lens=lens, need_v=False)
    many = [torch.full((binding.slim_workspace_bytes(B, H, T, H * d_k, "f32"),), 255, dtype=torch.uint8, device="cuda") for _ in range(16)]
    first = k.run_slim(workspace=many[0])
    assert k.err(first) <= TOL["f32"]
    assert np.array_equal(first, k.run_slim(workspace=many[1]))
    out = torch.empty((B, H * d_k), device="cuda")
    kw = dict(dtype="f32", seq_lens=k.lens_dev)

    def us(spaces):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for timed in (False, True):
            if timed:
                start.record()
            for i in range(96):
                binding.slim_decode(k.q, k.K, k.Wkv, out, B, H, T, H * d_k, workspace=spaces[i % len(spaces)], **kw)
        end.record()
        torch.cuda.synchronize()
        return start.elapsed_time(end) / 96 * 1e3

    us(many)
    t = [(us(many[:1]), us(many)) for _ in range(9)]
    one, turn = (statistics.median(x) for x in zip(*t))
    say(f"  one workspace {one:.2f} us, 16 in turn {turn:.2f} us")
    assert turn <= 1.06 * one
