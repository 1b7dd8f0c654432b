"""The wide K-cache path where scores are no ordinary numbers: whole 64-row blocks, whole context splits and whole sequences of -inf,
one +inf, one NaN, a sequence of length 0, and NaN in the rows past a sequence's end; with numerators per block and, heads of 8
columns, with the scores in their place.  What is finite agrees with the same in 64 bits (5e-5, as in test_gpu_wide_blocks.py);
what is not is NaN, and stays in its head."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding
from gpu_harness import say

pytestmark = pytest.mark.gpu

B, T = 5, 700


def _problem(d):
    import torch
    g = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn((B, d), generator=g, device="cuda") * 2
    K = torch.randn((B, T, d), generator=g, device="cuda").to(torch.bfloat16)
    W = (torch.randn((d, d), generator=g, device="cuda") * d ** -0.5).to(torch.bfloat16)
    return q, K, W


def _pull(q, K, d_k, b, h, signs):
    """Head h of sequence b: scores of `signs` (T,) times infinity, 0 where the sign is 0.  (3e38 x 1024 is past 32 bits.)"""
    q[b, h * d_k:(h + 1) * d_k] = 0
    q[b, h * d_k] = 3e38
    K[b, :len(signs), h * d_k] = (signs * 1024).to(K.dtype)


def _reference(q, K, W, lens, H):
    """In 64 bits, with the scores that overflow 32 bits as infinities; NaN where a head has a NaN or +inf score or no finite one."""
    import torch
    d = q.shape[1]
    d_k = d // H
    ref = torch.full((B, d), float("nan"), dtype=torch.float64, device="cuda")
    for b, n in enumerate(lens):
        if n == 0:
            continue
        rows = K[b, :n].double()
        s = (rows.view(n, H, d_k) * q[b].double().view(H, d_k)).sum(-1).T.contiguous() / d_k ** 0.5
        s[s > 3.4e38 / 1.4427] = float("inf")
        s[s < -3.4e38 / 1.4427] = float("-inf")
        full = torch.softmax(s, dim=1) @ rows @ W.double()
        ref[b] = full.view(H, H, d_k)[range(H), range(H)].reshape(d)
    return ref.cpu().numpy()


@pytest.mark.parametrize("H,d_k", [(40, 128), (48, 8)])
def test_scores_that_are_no_ordinary_numbers(H, d_k):
    import torch
    d = H * d_k
    q, K, W = _problem(d)
    lens = [700, 577, 0, 64, 700]
    lens_dev = torch.tensor(lens, dtype=torch.int32, device="cuda")
    t = torch.arange(T, device="cuda")
    minus, zero = -torch.ones(T, device="cuda"), torch.zeros(T, device="cuda")
    _pull(q, K, d_k, 0, 0, torch.where(t < 64, minus, zero))              # the first block -inf
    _pull(q, K, d_k, 0, 1, torch.where(t < 640, minus, zero))             # all splits but the last
    _pull(q, K, d_k, 0, 2, torch.where(t == 333, zero, minus))            # one row counts
    _pull(q, K, d_k, 0, 39, torch.where(t % 2 == 0, minus, zero))         # every second row
    _pull(q, K, d_k, 1, 7, torch.where(t < 560, zero, minus))             # the last, partial tile
    _pull(q, K, d_k, 3, 33, minus)                                        # no finite score: NaN
    _pull(q, K, d_k, 4, 5, torch.where(t == 100, -minus, zero))           # one +inf: NaN
    q[4, 20 * d_k + 3] = float("nan")                                     # NaN in a query: its head
    K[1, 577:] = float("nan")                                             # past the end
    K[3, 64:] = float("nan")
    ref = _reference(q, K, W, lens, H)
    outs = []
    for _ in range(2):
        say(f"[case] wide K-cache, extreme scores, {H} heads x {d_k}")
        out = torch.zeros((B, d), device="cuda")
        binding.slim_decode(q, K, W, out, B, H, T, d, seq_lens=lens_dev)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy().reshape(B, H, d_k).astype(np.float64))
    r = ref.reshape(B, H, d_k)
    lost = {(2, h) for h in range(H)} | {(3, 33), (4, 5), (4, 20)}
    assert {(b, h) for b in range(B) for h in range(H) if np.isnan(r[b, h]).any()} == lost
    for o in outs:
        nan = {(b, h) for b in range(B) for h in range(H) if np.isnan(o[b, h]).any()}
        part = {(b, h) for b, h in nan if not np.isnan(o[b, h]).all()}
        worst = max((float(np.abs(o[b, h] - r[b, h]).max() / np.abs(r[b, h]).max()), b, h) for b in range(B) for h in range(H) if (b, h) not in lost | nan)
        say(f"  NaN too many {sorted(nan - lost)}, missing {sorted(lost - nan)}, in part {sorted(part)}, worst of the others {worst}")
        assert nan == lost and not part and worst[0] <= 5e-5
    assert np.array_equal(outs[0], outs[1], equal_nan=True)
