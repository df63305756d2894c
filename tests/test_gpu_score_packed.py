"""GPU parity of the sweeps where the text queries of a q head are packed to sub-blocks of 16 rows: heads of one to nine sub-blocks, last
sub-blocks of one row and of sixteen, tiles that hold up to four heads or end inside one, last tiles past the last row, with queries
inside the video (whose mask then changes inside a tile).  test_launches.py asserts that they are.  Bounds: those of every score test."""
import pytest

import test_gpu_prune as base
import test_gpu_score_small as small

pytestmark = pytest.mark.gpu
B = base.B

# (layers, V, L, P, hq, hkv, d, mode), blocks of 256 rows a kv head
PACKED = [((2, 300, 1, 0, 28, 4, 128, 0), 1), ((2, 513, 17, 2, 7, 1, 64, 1), 1), ((2, 700, 28, 0, 64, 8, 128, 0), 1), ((2, 300, 32, 0, 5, 1, 64, 0), 1),
          ((2, 300, 16, 0, 17, 1, 64, 0), 2), ((12, 700, 33, 0, 20, 4, 64, 0), 1), ((12, 1300, 65, 0, 6, 2, 64, 0), 1), ((3, 2600, 100, 0, 16, 2, 64, 0), 4),
          ((16, 1300, 130, 0, 3, 1, 64, 0), 2), ((12, 2600, 33, 0, 5, 1, 128, 0), 1), ((16, 700, 80, 0, 6, 2, 128, 0), 1)]
# (V, L, first query's position, hq, hkv, d)
INSIDE = [(300, 24, 270, 9, 3, 64), (513, 17, 0, 10, 2, 64), (700, 30, 650, 16, 2, 128), (257, 1, 64, 27, 9, 128), (130, 16, 60, 21, 3, 64)]


@pytest.mark.parametrize("shape", [s for s, _ in PACKED])
def test_packed_rows(B, shape):
    base.test_score_layers_is_the_sum_over_layers(B, *shape)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("V,L,pos0,hq,hkv,d", INSIDE)
def test_packed_rows_inside_the_video(B, V, L, pos0, hq, hkv, d, mode):
    small.test_queries_inside_the_video(B, V, L, pos0, hq, hkv, d, mode)
