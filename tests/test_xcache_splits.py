"""Into how many context splits the one-pass X-cache kernel cuts a call: counts within 2 % of the best one that was measured, over widths and head
counts whose steps cost a quarter to all of the longest, and batches that an even share of the compute units does not hold."""
import pytest

from launch_rules import one_pass_cut, one_pass_splits


@pytest.mark.parametrize("B,H,T,d_model,best", [
    (64, 16, 1500, 512, (5, 6, 7)),                # narrow steps, the memory's rate: more than fill the chip once only add partials
    (27, 16, 1500, 512, (6, 7, 8, 9, 10)),
    (32, 16, 1500, 1024, (5, 6)),
    (12, 24, 1500, 896, (10, 12)),                 # two head tiles
    (13, 32, 1500, 640, (8, 9)),                   # one head tile in a workgroup (below), as the next: 31.2 us, 12 splits of two tiles 32.5
    (2, 128, 2290, 640, (11, 12, 13, 14, 15)),     # 32 to 33 us, 15 splits of two tiles 34.2
    (27, 40, 1500, 1280, (2,)),                    # three would take two rounds on some XCDs
    (7, 40, 1500, 1152, (10,)),
    (40, 128, 1500, 768, (3,)),                    # more than one round in any case
    (36, 128, 1355, 1024, (2, 3)),
    (8, 128, 4096, 1024, (8,)),
    (24, 20, 1500, 1280, (5,)),
])
def test_counts_that_were_measured(B, H, T, d_model, best):
    assert one_pass_splits(B, H, T, d_model)[0] in best


@pytest.mark.parametrize("d_model", range(512, 1281, 128))
def test_counts_stay_within_the_workspace(d_model):
    for B in (1, 3, 8, 31, 64, 300):
        for H in (1, 16, 17, 40, 128):
            for T in (1, 31, 128, 129, 1500, 4096, 70000):
                splits, most = one_pass_splits(B, H, T, d_model)
                assert 1 <= splits <= most <= 64


@pytest.mark.parametrize("B,H,T,d_model,best", [   # lengths from 100 to T
    (44, 128, 2655, 768, (2, 3, 4)),               # one split: 149 us, these 119 to 120
    (58, 128, 4437, 512, (3, 4, 5)),               # one: 187, these 155 to 157
    (53, 40, 3637, 640, (5, 6)),                   # two: 111, these 93 to 94
    (53, 20, 2515, 1280, (5,)),                    # two: 99, five 87
    (92, 40, 1661, 1024, (3,)),                    # one: 116, three 106
    (16, 64, 4694, 512, (8,)),                     # one round of workgroups, as if all had T rows
])
def test_counts_of_ragged_batches_that_were_measured(B, H, T, d_model, best):
    assert one_pass_splits(B, H, T, d_model, ragged=True)[0] in best


@pytest.mark.parametrize("B,H,T,d_model,tiles", [  # us with one head tile and with two
    (2, 32, 490, 1024, 1),                         # 24.9, 27.8
    (6, 64, 14, 1024, 1),                          # 21.9, 23.8
    (1, 64, 2998, 640, 1),                         # 28.4, 30.7
    (7, 64, 1654, 896, 1),                         # 33.6, 35.9
    (18, 128, 2145, 640, 2),                       # 84.9, 65.7
    (81, 64, 686, 512, 2),                         # 59.2, 55.3: two workgroups of one tile on a compute unit
    (80, 128, 1405, 512, 2),                       # 141.1, 136.4
    (8, 128, 4096, 1024, 2),
    (24, 20, 1500, 1280, 1),                       # (two do not fit)
    (8, 16, 4096, 1024, 1),
])
def test_head_tiles_that_were_measured(B, H, T, d_model, tiles):
    assert one_pass_cut(B, H, T, d_model)[0] == tiles
