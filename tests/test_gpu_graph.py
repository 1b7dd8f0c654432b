"""The decode calls recorded into a HIP graph: every replay, with new inputs and the program's own eager work between the
replays, gives the bits that an eager call gives on these inputs."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import BlockCase, KCase, XCase, say

pytestmark = pytest.mark.gpu
BASE = synth.CONFIGS[1]


def _replays(x, out, call):
    """x: the input tensor that changes from replay to replay; call(workspace or None): the call on x and out."""
    import torch
    binding.slim_init()
    first = x.clone()
    stream = torch.cuda.Stream()
    call(eager=True)                                     # (on another stream than the one that records)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call(eager=False)
    for i in range(5):
        x.copy_(first * (1.0 + 0.5 * i) if i % 2 else first.flip(-1) * (1.0 - 0.1 * i))
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        out.fill_(float("nan"))
        call(eager=True)
        torch.cuda.synchronize()
        assert torch.isfinite(out).all()
        assert torch.equal(got, out), f"replay {i}: {int((got != out).sum())} of {out.numel()} differ"


K_CASES = [  # (B, H, d_k, T, len_lo, dtype, banded, variant, static scratch)
    (1, 16, 128, 777, 0, "bf16", False, 0, True), (2, 20, 64, 700, 90, "bf16", False, 0, False), (3, 8, 96, 320, 10, "bf16", True, 0, True),
    (20, 8, 64, 300, 0, "bf16", False, 0, False), (1, 8, 64, 500, 0, "bf16", False, binding.VARIANT_FUSED_SPLIT, False),
    (2, 40, 64, 300, 20, "bf16", False, 0, False), (2, 8, 64, 300, 20, "f32", False, 0, True), (1, 8, 136, 100, 0, "bf16", False, 0, False),
]


@pytest.mark.parametrize("i", range(len(K_CASES)))
def test_decode_replays_match_eager_calls(i):
    import torch
    B, H, d_k, T, lo, dtype, banded, variant, static = K_CASES[i]
    say(f"[case] graph, decode: B={B} H={H} d_k={d_k} T={T} {dtype} banded={banded} variant={variant} static={static}")
    cfg = synth.scaled(BASE, B=B, H=H, d=H * d_k, d_k=d_k, T=T, len_lo=lo, dtype=dtype)
    k = KCase(cfg, q_scale=4.0, need_v=False, oracle_seqs={0}, t_stride=(T + 31) // 32 * 32)
    out = torch.empty((B, cfg.d), device="cuda", dtype=torch.float32)
    kw = dict(dtype=dtype, t_stride=k.t_stride, variant=variant, k_layout=binding.K_BANDED if banded else binding.K_ROWMAJOR,
              seq_lens=k.lens_dev if lo else None)
    K = k.banded_cache() if banded else k.K
    ws = [torch.empty(binding.slim_workspace_bytes(B, H, T, cfg.d, dtype), dtype=torch.uint8, device="cuda") for _ in range(2)]

    def call(eager):
        if static and not eager:
            binding.slim_decode_static(k.q, K, k.Wkv, out, B, H, T, cfg.d, **kw)
        else:
            binding.slim_decode(k.q, K, k.Wkv, out, B, H, T, cfg.d, workspace=ws[eager], **kw)
    _replays(k.q, out, call)


@pytest.mark.parametrize("d_model", [512, 384])
def test_xcache_replays_match_eager_calls(d_model):
    import torch
    say(f"[case] graph, X-cache: d_model={d_model}")
    cfg = synth.scaled(synth.CONFIGS[4], B=3, H=20, d=d_model, d_k=32, T=200)
    x = XCase(cfg, oracle_seqs={0})
    out = torch.empty((3, cfg.e), device="cuda", dtype=torch.float32)
    ws = [torch.empty(binding.slim_workspace_bytes_xcache(3, 20, 200, d_model, 32, "bf16"), dtype=torch.uint8, device="cuda") for _ in range(2)]
    _replays(x.q, out, lambda eager: binding.slim_decode_xcache(x.q, x.X, x.Wk, x.Wv, out, 3, 20, 200, d_model, 32, dtype="bf16", workspace=ws[eager]))


@pytest.mark.parametrize("vanilla", [False, True])
@pytest.mark.parametrize("B", [2, 18])
def test_block_replays_match_eager_calls(B, vanilla):
    import torch
    say(f"[case] graph, block: B={B} vanilla={vanilla}")
    cfg = synth.scaled(BASE, B=B, H=8, d=512, d_k=64, T=150, len_lo=20)
    b = BlockCase(cfg, rope_base=10000.0)
    y = torch.empty((B, 512), device="cuda", dtype=torch.float32)
    ws = [torch.empty(binding.slim_workspace_bytes_block(B, 8, 150, 512, "bf16"), dtype=torch.uint8, device="cuda") for _ in range(2)]

    def call(eager):
        if vanilla:
            binding.vanilla_attention_block(b.x, b.Wq, b.Wk, b.Wv, b.Wo, b.K_rot, b.V, y, B, 8, 150, 512, **b._kw(workspace=ws[eager]))
        else:
            binding.slim_attention_block(b.x, b.Wq, b.Wk, b.Wkv, b.Wo, b.K, y, B, 8, 150, 512, **b._kw(workspace=ws[eager]))
    _replays(b.x, y, call)
