"""GPU parity of the products where their loads of W are nontemporal, which one batch chunk of a large matrix has: a block's (one
sequence; with 17 there are two chunks, and the loads are ordinary), a wide layer's projection with one, two and four batch tiles,
and q~ and projection of an X-cache, whose every row is in use if no lengths are given."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import BlockCase, TOL, head_rel_err, row_rel_err, say
from launch_rules import batch_chunks, batch_tiles, read_once, xcache_read_once

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 17])
def test_products_of_large_matrices(B):
    say(f"[case] products of large matrices B={B}")
    cfg = synth.scaled(synth.CONFIGS[1], B=B, H=28, d=3584, d_k=128, T=20, len_lo=3)
    assert read_once(4 * 2 * cfg.d ** 2, 0)
    assert [batch_chunks(B, cfg.d, cfg.d, cfg.H * n) for n in (1, 2, 3)] == [1 if B == 1 else 2] * 3
    k = BlockCase(cfg)
    y, krow = k.run_slim()
    assert row_rel_err(y, k.ref) <= TOL["bf16"] and row_rel_err(krow, k.k_new) <= TOL["bf16"]
    assert np.array_equal(y, k.run_slim()[0])
    y, krow, vrow = k.run_vanilla()
    assert row_rel_err(y, k.ref) <= TOL["bf16"] and row_rel_err(krow, k.k_new) <= TOL["bf16"] and row_rel_err(vrow, k.v_new) <= TOL["bf16"]


def _weighted_rows(scores, rows):
    """scores (H, n), rows (n, w) -> (H, w): every head's softmax-weighted sum of the rows, in 64 bits."""
    import torch
    return torch.softmax(scores, dim=1) @ rows


@pytest.mark.parametrize("B,tiles", [(3, 1), (17, 2), (33, 4)])
def test_projection_of_a_wide_layer(B, tiles):
    import torch
    H, d_k, T = 56, 128, 40
    d = H * d_k
    assert read_once(2 * d * d, 0) and batch_tiles(B, d, d, H) == tiles and batch_chunks(B, d, d, H) == 1
    say(f"[case] projection of a wide layer B={B}")
    g = torch.Generator(device="cuda").manual_seed(B)
    q = torch.randn((B, d), generator=g, device="cuda") * 2
    K = torch.randn((B, T, d), generator=g, device="cuda").to(torch.bfloat16)
    W = (torch.randn((d, d), generator=g, device="cuda") * d ** -0.5).to(torch.bfloat16)
    lens = torch.tensor([T - b % 7 * 6 for b in range(B)], dtype=torch.int32, device="cuda")
    ref = torch.empty((B, d), device="cuda", dtype=torch.float64)
    W64 = W.double()
    for b in range(B):
        rows = K[b, :int(lens[b])].double()
        scores = (rows.view(-1, H, d_k) * q[b].double().view(H, d_k)).sum(-1).T.contiguous() / d_k ** 0.5
        full = _weighted_rows(scores, rows) @ W64
        ref[b] = full.view(H, H, d_k)[range(H), range(H)].reshape(d)
    out = [torch.empty((B, d), device="cuda") for _ in range(2)]
    for o in out:
        binding.slim_decode(q, K, W, o, B, H, T, d, seq_lens=lens)
    torch.cuda.synchronize()
    e = head_rel_err(out[0].cpu().numpy(), ref.cpu().numpy(), H)
    say(f"  rel err {e:.3e}")
    assert e <= 5e-5                   # fp32 but for the projection's split of C into two bf16 terms, 2^-17 per term
    assert torch.equal(out[0], out[1])


def test_xcache_weights():
    """Every row in use, once said by no lengths (nontemporal loads) and once by lengths of T: the same bits."""
    import torch
    B, H, d_k, T, d = 2, 128, 128, 8192, 1024
    e = H * d_k
    assert xcache_read_once(B, T, d, e, False, True) and not xcache_read_once(B, T, d, e, True, True)
    say("[case] X-cache, nontemporal weights")
    g = torch.Generator(device="cuda").manual_seed(1)
    q = torch.randn((B, e), generator=g, device="cuda")
    X = torch.randn((B, T, d), generator=g, device="cuda").to(torch.bfloat16)
    W_K, W_V = ((torch.randn((d, e), generator=g, device="cuda") * d ** -0.5).to(torch.bfloat16) for _ in range(2))
    out = [torch.empty((B, e), device="cuda") for _ in range(2)]
    binding.slim_decode_xcache(q, X, W_K, W_V, out[0], B, H, T, d, d_k)
    binding.slim_decode_xcache(q, X, W_K, W_V, out[1], B, H, T, d, d_k, seq_lens=torch.full((B,), T, dtype=torch.int32, device="cuda"))
    ref = torch.empty((B, e), device="cuda", dtype=torch.float64)
    for b in range(B):
        qt = torch.stack([W_K[:, h * d_k:(h + 1) * d_k].double() @ q[b, h * d_k:(h + 1) * d_k].double() for h in range(H)])
        C = _weighted_rows(qt @ X[b].double().T.contiguous() / d_k ** 0.5, X[b].double())
        ref[b] = torch.cat([C[h] @ W_V[:, h * d_k:(h + 1) * d_k].double() for h in range(H)])
    torch.cuda.synchronize()
    err = head_rel_err(out[0].cpu().numpy(), ref.cpu().numpy(), H)
    say(f"  rel err {err:.3e}")
    assert err <= TOL["bf16"]
    assert torch.equal(out[0], out[1])
