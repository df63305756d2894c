"""GPU parity of specvlm_score where the merge of the key splits changes shape: one block of rows is cut into one split per
64 keys, so 512 / 513 keys are the last launch with one lane per row and the first with eight, 4096 keys have the most
splits a row can have, 4097 half as many; with prefix rows, hidden text keys and keyless splits.  Bounds: those of
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
