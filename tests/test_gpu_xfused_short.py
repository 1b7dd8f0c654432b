"""The one-pass X-cache kernel on contexts of one tile of rows, which have a way of their own through it, beside ones of two, with head counts on
either side of a group (the partial's stores drop the heads that are not there): against the fp64 oracle, which sees the weights as stored, at the
tolerance of bf16 caches, the same bits twice, and nothing written past the workspace."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import TOL, XCase, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [5, 16, 17, 40])
@pytest.mark.parametrize("d", [512, 640, 768, 896, 1024, 1152, 1280])
def test_contexts_of_one_tile_match_oracle(d, H):
    import torch
    for B, T, lens in ((3, 1, None), (4, 33, [33, 32, 1, 17]), (9, 32, [32, 31, 9, 1, 16, 8, 32, 3, 2]), (70, 32, None)):
        cfg = synth.scaled(synth.CONFIGS[4], B=B, H=H, d=d, d_k=32, T=T)
        say(f"[case] short X-cache: B={B} H={H} d_model={d} T={T} lens={lens}")
        x = XCase(cfg, q_scale=4.0, lens=lens, oracle_seqs=None if B < 20 else {0, 35, 69}, oracle_sees_rounded_weights=True)
        need = binding.slim_workspace_bytes_xcache(B, H, T, d, 32, "bf16")
        ws = torch.full((need + 65536,), 0xA5, dtype=torch.uint8, device="cuda")
        a = x.run(workspace=ws[:need])
        e = x.err(a)
        say(f"  rel err {e:.3e}")
        assert e <= TOL["bf16"]
        assert bool((ws[need:] == 0xA5).all())
        assert np.array_equal(a, x.run())
