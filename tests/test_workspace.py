"""A workspace sized for the longest context serves every shorter one: the sizes never shrink as T grows.  CPU only."""
import random

import pytest

from paper_2503_05840_amd import binding

T_STEPS = sorted({t for k in range(0, 16) for t in (2 ** k - 1, 2 ** k, 2 ** k + 1) if t > 0} | set(range(1, 300, 7)) |
                 set(range(224, 9000, 32)) | set(range(6001, 7000, 71)) | set(range(9000, 70000, 509)))


def _never_shrinks(size):
    last, at = 0, 0
    for T in T_STEPS:
        n = size(T)
        assert n >= last, f"{n} bytes at T = {T}, {last} at T = {at}"
        last, at = n, T


@pytest.mark.parametrize("B,H,d_k,d_model", [(24, 128, 128, 1024), (32, 40, 32, 1280), (1, 8, 64, 512), (100, 12, 64, 768), (7, 33, 32, 2048)])
def test_xcache_workspace_never_shrinks_with_the_context(B, H, d_k, d_model):
    _never_shrinks(lambda T: binding.slim_workspace_bytes_xcache(B, H, T, d_model, d_k, "bf16"))


@pytest.mark.parametrize("B,H,d_k", [(32, 40, 32), (24, 12, 96), (1, 8, 64), (4, 16, 64), (16, 32, 96), (64, 20, 64), (200, 32, 32), (1, 1, 1024)])
def test_kcache_and_block_workspaces_never_shrink_with_the_context(B, H, d_k):
    _never_shrinks(lambda T: binding.slim_workspace_bytes(B, H, T, H * d_k, "bf16"))
    _never_shrinks(lambda T: binding.slim_workspace_bytes_block(B, H, T, H * d_k, "bf16"))


def test_workspaces_of_random_shapes_never_shrink_with_the_context():
    rng = random.Random(5)
    for _ in range(60):
        B, H, d_k = int(2 ** rng.uniform(0, 9)), rng.randint(1, 130), 8 * rng.randint(1, 32)
        d_model = rng.choice([64, 256, 384, 512, 640, 768, 896, 1024, 1152, 1280, 2048])
        try:
            _never_shrinks(lambda T: binding.slim_workspace_bytes(B, H, T, H * d_k, "f32"))
            _never_shrinks(lambda T: binding.slim_workspace_bytes_xcache(B, H, T, d_model, d_k, "bf16"))
        except AssertionError as e:
            raise AssertionError(f"B = {B}, H = {H}, d_k = {d_k}, d_model = {d_model}") from e
