"""GPU parity of specvlm_score's two-launch form for one small layer: up to eight row tiles (64 text queries of a q head)
over up to 17408 keys.  Tiles with one to all live queries, one and more tiles a head, one and more kv heads, last key
ranges and last columns that are not full, prefix rows, hidden keys, more key ranges than a row has visible keys; and the
first shapes beyond it (nine tiles, 17409 keys), which the sweeps still take, with their splits on both sides of eight.
Bounds: those of every score test."""
import numpy as np
import pytest

import oracle
import test_gpu_prune as base
from gpu_util import dev_bf16, rnd_bits
from test_gpu_prune import assert_scores_close

pytestmark = pytest.mark.gpu
B = base.B


@pytest.mark.parametrize("V,L,P,hq,hkv,d,mode", [
    (1568, 64, 0, 4, 1, 64, 0), (1, 1, 0, 1, 1, 64, 0), (63, 63, 0, 4, 2, 64, 1), (64, 64, 0, 8, 1, 128, 0),
    (65, 65, 3, 4, 4, 64, 0), (300, 130, 0, 2, 1, 128, 1), (700, 512, 9, 1, 1, 64, 0), (2100, 17, 0, 8, 8, 64, 0),
    (1000, 1, 2000, 3, 1, 128, 0), (17343, 64, 1, 2, 2, 64, 0), (17344, 64, 1, 2, 2, 64, 0), (500, 64, 0, 9, 1, 64, 0),
    (430, 64, 0, 9, 1, 64, 0), (4032, 64, 0, 9, 1, 64, 0), (700, 64, 0, 6, 1, 64, 0),      # (the last: 58 KB of LDS)
])
def test_small_layer(B, V, L, P, hq, hkv, d, mode):
    base.test_score_matches_oracle(B, V, L, P, hq, hkv, d, mode)
    base.test_score_layers_is_the_sum_over_layers(B, 1, V, L, P, hq, hkv, d, mode)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("V,L,pos0,hq,hkv,d", [(300, 40, 270, 4, 2, 64), (200, 100, 0, 2, 1, 128), (130, 64, 64, 8, 1, 64)])
def test_queries_inside_the_video(B, V, L, pos0, hq, hkv, d, mode):
    """Text queries that stand inside the video span, head-major keys, and beta on top of what was there."""
    q, k = rnd_bits((L, hq, d), 160), rnd_bits((V + L, hkv, d), 161)
    before = np.linspace(0.0, 1.0, V).astype(np.float32)
    want = oracle.score(q, k, 0, V, pos0, 0.125, norm_mode=mode, beta=0.5, scores_in=before)
    kd = dev_bf16(k.transpose(1, 0, 2)).permute(1, 0, 2)
    got = B.score(dev_bf16(q), kd, 0, V, pos0, 0.125, norm_mode=mode, beta=0.5, scores=base.torch.from_numpy(before).cuda())
    base.torch.cuda.synchronize()
    assert_scores_close(got, want, f"V{V} L{L} pos0 {pos0} mode{mode}")


def test_key_that_towers_over_all_others_and_zero_scale(B):
    V, L, hq, hkv, d = 1300, 33, 4, 1, 64
    q, k = rnd_bits((L, hq, d), 260), rnd_bits((V + L, hkv, d), 261)
    k[700] = rnd_bits((hkv, d), 262, 60.0)
    for scale in (0.125, 0.0):
        want = oracle.score(q, k, 0, V, V, scale)
        got = B.score(dev_bf16(q), dev_bf16(k), 0, V, V, scale)
        base.torch.cuda.synchronize()
        assert_scores_close(got, want, f"scale {scale}")
