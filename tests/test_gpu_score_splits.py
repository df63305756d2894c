"""GPU parity of specvlm_score where its merges change shape.  Key counts on both sides of 8 and 64 times 64, with prefix rows
and hidden text keys: one layer of so few rows takes the two-launch form, which cuts them into up to 32 key ranges (the sweeps'
splits of such counts: test_gpu_score_sweeps.py).  Partial columns of the sweeps: up to sixteen of them (layers x kv heads x row
splits) one thread sums a column, with eight or sixteen loads, then eight threads; one layer of 9 and 16 heads (5 and 8 take
the two-launch form) with one row split each, 2 and 17 layers of one head, columns that do not fill the last workgroup.  Bounds: those of
every score test."""
import pytest

import test_gpu_prune as base

pytestmark = pytest.mark.gpu
B = base.B


@pytest.mark.parametrize("V,L,P,hq,hkv,d,mode", [
    (496, 16, 0, 4, 1, 64, 0), (497, 16, 0, 4, 1, 64, 0), (512, 3, 0, 4, 1, 64, 1), (513, 3, 7, 4, 1, 64, 1),
    (4080, 16, 0, 2, 1, 128, 0), (4081, 16, 0, 2, 1, 128, 0), (40, 1, 0, 1, 1, 64, 0),
])
def test_key_splits(B, V, L, P, hq, hkv, d, mode):
    base.test_score_matches_oracle(B, V, L, P, hq, hkv, d, mode)


@pytest.mark.parametrize("layers,V,L,P,hq,hkv,d,mode", [
    (1, 4100, 5, 0, 5, 5, 64, 0), (1, 300, 5, 0, 8, 8, 64, 0), (1, 300, 5, 0, 9, 9, 64, 0), (1, 2049, 3, 0, 16, 16, 64, 0), (2, 33, 3, 0, 1, 1, 64, 0), (17, 257, 4, 2, 1, 1, 64, 1),
    (3, 1, 2, 0, 8, 2, 128, 0),
])
def test_partial_columns(B, layers, V, L, P, hq, hkv, d, mode):
    base.test_score_layers_is_the_sum_over_layers(B, layers, V, L, P, hq, hkv, d, mode)


# sixteen partial columns are the last that one thread sums: one row split each, layers x heads on both sides of the line
@pytest.mark.parametrize("layers,V,L,P,hq,hkv,d,mode", [
    (2, 300, 5, 0, 8, 8, 64, 0), (1, 2049, 3, 0, 17, 17, 64, 0), (16, 257, 4, 0, 1, 1, 64, 1), (3, 4100, 3, 2, 5, 5, 64, 0),
    (2, 270, 40, 0, 14, 2, 64, 0), (5, 255, 3, 0, 6, 3, 128, 0),
])
def test_partial_columns_of_one_thread(B, layers, V, L, P, hq, hkv, d, mode):
    base.test_score_layers_is_the_sum_over_layers(B, layers, V, L, P, hq, hkv, d, mode)
