"""How the one-pass X-cache kernel cuts a call: context splits, on whose count the rounding of its results depends and which stay what they are, and the
heads of a workgroup."""
import pytest

from launch_rules import one_pass_splits, one_pass_tiles

SPLITS = [  # (B, H, T, d_model, count)
    (8, 128, 4096, 1024, 8), (24, 20, 1500, 1280, 5), (64, 16, 1500, 1024, 4), (32, 16, 1500, 1024, 8),
    (64, 16, 1500, 512, 8), (27, 40, 1500, 1280, 3), (3, 64, 2290, 640, 18), (13, 32, 1500, 640, 8),
    (40, 128, 1500, 768, 1), (55, 40, 7576, 512, 2), (1, 128, 300, 1024, 3), (12, 24, 1500, 896, 8),
    (7, 40, 1500, 1152, 8), (1, 8, 100, 512, 1),
]


@pytest.mark.parametrize("B,H,T,d_model,splits", SPLITS)
def test_counts_stay_what_they_are(B, H, T, d_model, splits):
    assert one_pass_splits(B, H, T, d_model)[0] == splits


@pytest.mark.parametrize("B,H,T,d_model,tiles", [  # us with one head tile and with two
    (2, 32, 490, 1024, 1),                         # 24.9, 27.8
    (6, 64, 14, 1024, 1),                          # 21.9, 23.8
    (1, 64, 2998, 640, 1),                         # 28.4, 30.7
    (18, 128, 2145, 640, 2),                       # 84.9, 65.7
    (81, 64, 686, 512, 2),                         # 59.2, 55.3: two workgroups of one tile on a compute unit
    (80, 128, 1405, 512, 2),                       # 141.1, 136.4
    (8, 128, 4096, 1024, 2),
    (24, 20, 1500, 1280, 1),                       # (two do not fit)
    (8, 16, 4096, 1024, 1),
])
def test_head_tiles_that_were_measured(B, H, T, d_model, tiles):
    assert one_pass_tiles(B, H, T, d_model) == tiles


@pytest.mark.parametrize("d_model", range(512, 1281, 128))
def test_counts_stay_within_the_workspace(d_model):
    for B in (1, 3, 8, 31, 64, 300):
        for H in (1, 16, 17, 40, 128):
            for T in (1, 31, 128, 129, 1500, 4096, 70000):
                splits, most = one_pass_splits(B, H, T, d_model)
                assert 1 <= splits <= most <= 64
