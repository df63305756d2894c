"""GPU parity of specvlm_score's sweeps at the edges of their merges and masks, with shapes that the two-launch form of one small
layer does not take: two layers or more, or nine row tiles (64 text queries of a q head) and more.  Which kernels
serve them, with how many splits and partial columns, is asserted in test_launches.py.  Bounds: those of every score test."""
import pytest

import test_gpu_prune as base
import test_gpu_score_small as small

pytestmark = pytest.mark.gpu
B = base.B

# two layers of one block of rows, one key split per 64 keys: (V, L, P, hq, hkv, d, mode), splits.  Eight are the last launch with
# one lane per row and nine the first with eight, 64 the most that a row can have, one key more half as many.
KEY_SPLITS = [
    ((496, 16, 0, 4, 1, 64, 0), 8), ((497, 16, 0, 4, 1, 64, 0), 9), ((512, 3, 7, 4, 1, 64, 1), 8), ((513, 3, 7, 4, 1, 64, 1), 9),
    ((489, 16, 7, 2, 1, 128, 0), 8), ((490, 16, 7, 2, 1, 128, 0), 9), ((512, 5, 0, 4, 1, 128, 1), 8), ((513, 5, 0, 4, 1, 128, 1), 9),
    ((4080, 16, 0, 2, 1, 128, 0), 64), ((4081, 16, 0, 2, 1, 128, 0), 33), ((4096, 5, 9, 4, 1, 64, 1), 64), ((4097, 5, 9, 4, 1, 64, 1), 33),
    ((4096, 5, 9, 2, 1, 128, 1), 64), ((4070, 17, 9, 4, 1, 64, 0), 64), ((40, 1, 0, 1, 1, 64, 0), 1),
]


@pytest.mark.parametrize("shape,splits", KEY_SPLITS)
def test_key_splits(B, shape, splits):
    base.test_score_layers_is_the_sum_over_layers(B, 2, *shape)


# (layers, V, L, P, hq, hkv, d, mode), partial columns (one row split each): eight are the last that one thread sums with eight
# loads, sixteen the last that one thread sums at all
PARTIAL_COLUMNS = [((2, 300, 5, 0, 4, 4, 64, 0), 8), ((8, 300, 5, 2, 1, 1, 128, 1), 8), ((3, 300, 5, 0, 3, 3, 64, 0), 9), ((2, 700, 9, 0, 8, 8, 64, 1), 16),
                   ((1, 300, 5, 0, 9, 9, 64, 0), 9), ((17, 257, 4, 0, 1, 1, 64, 0), 17)]


@pytest.mark.parametrize("shape,columns", PARTIAL_COLUMNS)
def test_partial_columns(B, shape, columns):
    base.test_score_layers_is_the_sum_over_layers(B, *shape)


# (V, L, first query's position, hq, hkv, d): last video blocks that are not full, waves of padding only in them and in the rows
INSIDE = [(300, 40, 270, 9, 3, 64), (513, 100, 0, 10, 2, 64), (700, 70, 650, 8, 2, 128), (257, 64, 64, 16, 1, 128), (1300, 130, 600, 28, 4, 128),
          (65, 65, 1, 9, 9, 64)]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("V,L,pos0,hq,hkv,d", INSIDE)
def test_queries_inside_the_video(B, V, L, pos0, hq, hkv, d, mode):
    small.test_queries_inside_the_video(B, V, L, pos0, hq, hkv, d, mode)


def test_logits_that_outgrow_the_earlier_tiles_at_head_size_64(B):
    base.test_score_logits_that_outgrow_the_earlier_tiles(B, 64, 10, 2)
