"""The one-pass X-cache kernel where its inputs are no ordinary numbers, in a cache with more rows than the call reads: tiles, context splits and
whole sequences of -inf scores, one +inf, one NaN, a sequence of length 0, NaN in the rows past a sequence's end and between T and t_stride.
What is finite agrees with the same in 64 bits at the tolerance of bf16 caches; what is not is NaN, and stays in its head."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding
from gpu_harness import TOL, say

pytestmark = pytest.mark.gpu

B, T, STRIDE, DK = 5, 700, 737, 32


def _reference(q, X, WK, WV, lens, H):
    """In 64 bits, with the scores that overflow 32 bits as infinities; NaN where a head has a NaN or +inf score or no finite one."""
    import torch
    ref = torch.full((B, H * DK), float("nan"), dtype=torch.float64, device="cuda")
    for b, n in enumerate(lens):
        if n == 0:
            continue
        rows = X[b, :n].double()
        for h in range(H):
            c = slice(h * DK, (h + 1) * DK)
            s = rows @ (WK[:, c].double() @ q[b, c].double()) / DK ** 0.5
            s[s > 3.4e38 / 1.4427] = float("inf")
            s[s < -3.4e38 / 1.4427] = float("-inf")
            ref[b, c] = (torch.softmax(s, dim=0) @ rows) @ WV[:, c].double()
    return ref.cpu().numpy().reshape(B, H, DK)


@pytest.mark.parametrize("H,d", [(20, 512), (40, 640), (20, 1024), (16, 1280)])
def test_scores_that_are_no_ordinary_numbers(H, d):
    import torch
    g = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    q, X = rnd(B, H * DK) * 2, rnd(B, STRIDE, d).to(torch.bfloat16)
    WK, WV = ((rnd(d, H * DK) * d ** -0.5).to(torch.bfloat16) for _ in range(2))
    t = torch.arange(T, device="cuda")
    minus, zero = -torch.ones(T, device="cuda"), torch.zeros(T, device="cuda")

    def pull(b, h, signs):
        """Head h of sequence b: scores of `signs` (T,) times infinity, 0 where the sign is 0, by a column of X that this head alone sees."""
        col = 3 + 29 * h % d
        WK[:, h * DK] = 0
        WK[col] = 0
        WK[col, h * DK] = 1
        q[:, h * DK] = 0
        q[b, h * DK:(h + 1) * DK] = 0
        q[b, h * DK] = 3e38                                               # (times 1024 it is past 32 bits)
        X[b, :T, col] = (signs * 1024).to(X.dtype)

    pull(0, 0, torch.where(t < 64, minus, zero))                          # the first tiles
    pull(0, 1, torch.where(t < 640, minus, zero))                         # all splits but the last
    pull(0, 2, torch.where(t == 333, zero, minus))                        # one row counts
    pull(0, 3, torch.where(t % 2 == 0, minus, zero))                      # every second row
    pull(1, 4, torch.where(t < 560, zero, minus))                         # the last, partial tile
    pull(3, 5, minus)                                                     # no finite score: NaN
    pull(4, 6, torch.where(t == 100, -minus, zero))                       # one +inf: NaN
    q[4, 7 * DK + 3] = float("nan")                                       # NaN in a query: its head
    lens = [700, 577, 0, 20, 700]
    for b, n in enumerate(lens):
        X[b, n:] = float("nan")
    ref = _reference(q, X, WK, WV, lens, H)
    lost = {(2, h) for h in range(H)} | {(3, 5), (4, 6), (4, 7)}
    assert {(b, h) for b in range(B) for h in range(H) if np.isnan(ref[b, h]).any()} == lost
    lens_dev = torch.tensor(lens, dtype=torch.int32, device="cuda")
    outs = []
    for _ in range(2):
        say(f"[case] one-pass X-cache, extreme scores: H={H} d_model={d} T={T} t_stride={STRIDE} lens={lens}")
        out = torch.zeros((B, H * DK), device="cuda")
        binding.slim_decode_xcache(q, X, WK, WV, out, B, H, T, d, DK, seq_lens=lens_dev, t_stride=STRIDE)
        torch.cuda.synchronize()
        outs.append(out.cpu().numpy().reshape(B, H, DK).astype(np.float64))
    for o in outs:
        nan = {(b, h) for b in range(B) for h in range(H) if np.isnan(o[b, h]).any()}
        part = {(b, h) for b, h in nan if not np.isnan(o[b, h]).all()}
        worst = max((float(np.abs(o[b, h] - ref[b, h]).max() / np.abs(ref[b, h]).max()), b, h) for b in range(B) for h in range(H) if (b, h) not in lost | nan)
        say(f"  NaN too many {sorted(nan - lost)}, missing {sorted(lost - nan)}, in part {sorted(part)}, worst of the others {worst}")
        assert nan == lost and not part and worst[0] <= TOL["bf16"]
    assert np.array_equal(outs[0], outs[1], equal_nan=True)
