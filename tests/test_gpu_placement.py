"""Where the workgroups that share a result meet.  On a device that deals workgroups to the XCDs in turn they meet in an
XCD's L2; on others at the memory side: the same sums in the same order, so the results are the same bits.  Which XCD a
launch starts on differs from stream to stream.  The workgroups check that they share an XCD: with every second of them
behaving as if it did not (forced from the host; every kernel ends normally) the results are NaN and slim_status says so,
and the next ordinary call on the same scratch is clean again."""
import numpy as np
import pytest

from paper_2503_05840_amd import binding, synth
from gpu_harness import BlockCase, KCase, XCase, say

pytestmark = pytest.mark.gpu
BASE = synth.CONFIGS[1]
VIA_MEMORY, APART = binding.VARIANT_VIA_MEMORY, binding.VARIANT_APART

# (every case has rows of W for more than one workgroup)
K_CASES = [  # (B, H, d_k, T, variant)
    (1, 32, 128, 777, binding.VARIANT_AUTO), (3, 20, 64, 300, binding.VARIANT_AUTO), (2, 16, 80, 300, binding.VARIANT_AUTO),
    (16, 8, 128, 200, binding.VARIANT_AUTO), (1, 8, 64, 500, binding.VARIANT_FUSED_SPLIT), (20, 16, 48, 130, binding.VARIANT_AUTO),
    (64, 20, 64, 300, binding.VARIANT_AUTO), (2, 40, 64, 200, binding.VARIANT_AUTO),
]
X_CASES = [(3, 16, 512, 32, 300), (2, 40, 1024, 32, 200)]
BLOCKS = [(4, 16, 64, 200, None), (16, 8, 128, 130, 10000.0), (3, 8, 80, 100, None)]


def _every_way(run):
    """The call as the library makes it, by way of memory, on other streams, apart, and once more: lists of outputs."""
    import torch
    binding.slim_init()
    good = run(0)
    assert binding.slim_status(None) == binding.SLIM_OK
    for o in good:
        assert np.isfinite(o).all()
    for o, m in zip(good, run(VIA_MEMORY)):
        assert np.array_equal(o, m)
    assert binding.slim_status(None) == binding.SLIM_OK
    for _ in range(5):                                   # (more streams than hardware queues)
        with torch.cuda.stream(torch.cuda.Stream()):
            for o, m in zip(good, run(0)):
                assert np.array_equal(o, m)
            assert binding.slim_status(None) == binding.SLIM_OK
    bad = run(APART)
    assert binding.slim_status(None) == binding.SLIM_ERR_TIMEOUT
    for o in bad:
        assert np.isnan(o).all()
    for o, a in zip(good, run(0)):
        assert np.array_equal(o, a)
    assert binding.slim_status(None) == binding.SLIM_OK


@pytest.mark.parametrize("i", range(len(K_CASES)))
def test_decode_meets_in_l2_or_memory_and_notices_when_apart(i):
    B, H, d_k, T, variant = K_CASES[i]
    say(f"[case] placement, decode: B={B} H={H} d_k={d_k} T={T} variant={variant}")
    k = KCase(synth.scaled(BASE, B=B, H=H, d=H * d_k, d_k=d_k, T=T), need_v=False, oracle_seqs={0})
    _every_way(lambda f: [k.run_slim(variant=variant + f)])


@pytest.mark.parametrize("i", range(len(X_CASES)))
def test_xcache_meets_in_l2_or_memory_and_notices_when_apart(i):
    B, H, d, d_k, T = X_CASES[i]
    say(f"[case] placement, X-cache: B={B} H={H} d_model={d} d_k={d_k} T={T}")
    x = XCase(synth.scaled(synth.CONFIGS[4], B=B, H=H, d=d, d_k=d_k, T=T), oracle_seqs={0})
    _every_way(lambda f: [x.run(variant=f)])


@pytest.mark.parametrize("vanilla", [False, True])
@pytest.mark.parametrize("i", range(len(BLOCKS)))
def test_block_meets_in_l2_or_memory_and_notices_when_apart(i, vanilla):
    B, H, d_k, T, rope = BLOCKS[i]
    say(f"[case] placement, block: B={B} H={H} d_k={d_k} T={T} rope={rope} vanilla={vanilla}")
    b = BlockCase(synth.scaled(BASE, B=B, H=H, d=H * d_k, d_k=d_k, T=T), rope_base=rope)
    _every_way(lambda f: list(b.run_vanilla(variant=f) if vanilla else b.run_slim(variant=f)))
