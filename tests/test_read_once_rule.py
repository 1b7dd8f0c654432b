"""Which calls read their weights with nontemporal loads: only what a call is known to read counts towards the size from which
it pays, so never rows that a ragged batch may leave unused, and no cache that is read twice."""
import pytest

from launch_rules import batch_chunks, batch_tiles, read_once, xcache_read_once


@pytest.mark.parametrize("B,T,H,d,ragged,one_pass,want", [
    (8, 4096, 128, 1024, False, True, True),       # 134 MB for certain
    (8, 4096, 128, 1024, True, True, False),       # 67 MB of weights; of X it may be 400 rows of 4096
    (4, 4096, 128, 1024, False, True, True),       # 100.7 MB, on the line
    (4, 4095, 128, 1024, False, True, False),
    (16, 8192, 128, 1024, False, True, True),
    (8, 4096, 64, 1024, False, True, False),       # 34 MB of weights
    (8, 4096, 80, 1280, False, True, False),       # 52 MB of weights
    (4, 6000, 128, 2048, False, False, False),     # X is read a second time, from the memory-side cache
])
def test_xcache(B, T, H, d, ragged, one_pass, want):
    assert xcache_read_once(B, T, d, H * 128, ragged, one_pass) == want


@pytest.mark.parametrize("matrices,d,want", [
    (4, 4096, True), (4, 3584, True), (4, 3072, False),                # blocks
    (1, 8192, True), (1, 7168, True), (1, 5120, False), (1, 6144, False),      # wide layers: K is read twice and does not count
])
def test_weights_alone(matrices, d, want):
    assert read_once(matrices * 2 * d * d, 0) == want


def test_blocks_of_several_batch_tiles_come_in_several_chunks():
    """(the reason why a block's products have nontemporal loads with one batch tile only)"""
    for H in range(1, 33):                                             # what the block's fast path takes: 32 heads, 4096 columns
        for d_k in (8, 16, 32, 64, 72, 80, 96, 104, 112, 120, 128):
            d = H * d_k
            if d <= 4096 and read_once(4 * 2 * d * d, 0):
                for B in range(1, 1025):
                    for units in (H, 2 * H, 3 * H):
                        assert batch_tiles(B, d, d, units) == 1 or batch_chunks(B, d, d, units) > 1
