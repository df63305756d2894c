"""GPU parity of the decode attention over short caches where its workgroups go from eight waves to sixteen: the last cache
length of one and the first of the other, waves without keys and with a single one, launches that leave some, one or no CU
for helper workgroups, a ragged batch and a tree.  Bounds: those of every attention test."""
import pytest

import test_gpu_attn_short as base

pytestmark = pytest.mark.gpu
B = base.B


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d", [
    (1, 1280, 14, 2, 64), (1, 1281, 14, 2, 64), (3, 1344, 14, 2, 64), (2, 1345, 8, 8, 64), (16, 1441, 32, 8, 64),
    (1, 640, 8, 2, 128), (1, 641, 8, 2, 128), (8, 641, 64, 8, 128), (6, 705, 64, 8, 128), (4, 961, 32, 4, 128), (31, 700, 8, 4, 128),
    (1, 768, 8, 2, 128), (1, 769, 8, 2, 128), (8, 769, 64, 8, 128), (31, 800, 8, 4, 128),
])
def test_edges(B, q_len, kv_len, hq, hkv, d):
    base.test_edges_match_oracle(B, q_len, kv_len, hq, hkv, d, 0)


@pytest.mark.parametrize("lens,hq,hkv,d", [([1281, 1400, 33, 1536], 8, 2, 64), ([641, 3, 900], 8, 2, 128), ([641, 3, 768], 8, 2, 128)])
def test_ragged_batch(B, lens, hq, hkv, d):
    base.ragged_case(B, lens, [2] * len(lens), hq, hkv, d)


@pytest.mark.parametrize("n_nodes,kv_len,hq,hkv,d", [(26, 1400, 14, 2, 64), (40, 800, 4, 1, 128)])
def test_tree(B, n_nodes, kv_len, hq, hkv, d):
    base.test_tree_over_a_short_cache(B, n_nodes, kv_len, hq, hkv, d)


@pytest.mark.parametrize("kv_len,d", [(40, 64), (600, 64), (1400, 64), (33, 128), (500, 128), (900, 128)])
@pytest.mark.parametrize("q_len,hq,hkv", [(1, 1, 1), (5, 2, 2), (7, 1, 1), (4, 4, 2), (3, 3, 1), (5, 6, 2), (16, 2, 2), (17, 1, 1)])
def test_rows_of_a_block(B, q_len, hq, hkv, kv_len, d):
    """1 to 17 query rows a kv head: a row of a block is 16 lanes' work where the waves' results meet, the rows that are not there nobody's."""
    base.test_edges_match_oracle(B, q_len, kv_len, hq, hkv, d, 0)
