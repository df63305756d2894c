"""GPU parity of the decode-attention launches for short caches (no splits, no merge) and of the short key splits,
at the edges where their shapes change: chunk and wave ends, the last cache length of the launch and the first
beyond it, one and several row blocks, ragged batches, a tree, both layouts, keys that tower over all others.  Bounds: those of every attention test (max-abs 2e-2,
mean-abs 2e-3 for outputs of size one: bf16 in and out, fp32 sums)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_16201_amd import synth
from gpu_util import dev_bf16, host_f64, rnd_bits, assert_attn_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2508_16201_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d,splits", [
    (1, 2, 2, 2, 64, 0), (1, 33, 4, 1, 64, 0), (2, 255, 14, 2, 64, 0), (3, 256, 14, 2, 64, 0),   # 21 rows: two row blocks
    (1, 257, 4, 1, 64, 0), (6, 1023, 12, 3, 64, 0),                   # 3 kv heads: helpers and heads out of step
    (1, 1535, 14, 2, 64, 0), (2, 1536, 16, 2, 64, 0), (1, 1537, 14, 2, 64, 0),
    (1, 16, 8, 8, 128, 0), (5, 289, 32, 2, 128, 0), (4, 768, 8, 2, 128, 0), (6, 1024, 16, 2, 128, 0),
    (1, 1025, 7, 1, 128, 0), (8, 64, 64, 8, 128, 0),                  # 256 workgroups: the most without a second round
    (8, 65, 72, 8, 128, 0),                                           # 72 rows per kv head: splits
    (1, 500, 14, 2, 64, 4), (1, 500, 14, 2, 64, 5), (1, 2049, 4, 1, 64, 17),   # short splits: four of 125 keys (five are clamped), a last one of 113
])
def test_edges_match_oracle(B, q_len, kv_len, hq, hkv, d, splits):
    q, k, v = (rnd_bits((n, h, d), 5000 + kv_len + i) for i, (n, h) in enumerate(((q_len, hq), (kv_len, hkv), (kv_len, hkv))))
    scale = 1.0 / np.sqrt(d)
    want, want_lse = oracle.decode_attn(q, k, v, scale)
    out, lse = B.decode_attn(dev_bf16(q), dev_bf16(k), dev_bf16(v), scale, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    assert_attn_close(out, want, f"q{q_len} kv{kv_len} {hq}/{hkv} d{d} splits {splits}")
    np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4)


def ragged_case(B, lens, q_lens, hq, hkv, d, **more):
    q, k, v = [], [], []
    for i, (n, m) in enumerate(zip(lens, q_lens)):
        q.append(rnd_bits((m, hq, d), 5600 + i)); k.append(rnd_bits((n, hkv, d), 5700 + i)); v.append(rnd_bits((n, hkv, d), 5800 + i))
    cu = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32).cuda()  # noqa: E731
    out = B.decode_attn(dev_bf16(np.concatenate(q)), dev_bf16(np.concatenate(k)), dev_bf16(np.concatenate(v)), 0.125,
                        cu_q=cu(q_lens), cu_kv=cu(lens), max_q_len=max(q_lens), max_kv_len=max(lens), **more)
    torch.cuda.synchronize()
    o = 0
    for i, m in enumerate(q_lens):
        assert_attn_close(out[o:o + m], oracle.decode_attn(q[i], k[i], v[i], 0.125)[0], f"request {i}")
        o += m


def test_ragged_batch_of_short_caches(B):
    lens, q_lens, hq, hkv, d = [1500, 3, 257, 1024, 64], [1, 3, 2, 3, 1], 14, 2, 64
    q, k, v = [], [], []
    for i, (n, m) in enumerate(zip(lens, q_lens)):
        q.append(rnd_bits((m, hq, d), 5600 + i)); k.append(rnd_bits((n, hkv, d), 5700 + i)); v.append(rnd_bits((n, hkv, d), 5800 + i))
    cu = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32).cuda()  # noqa: E731
    out = B.decode_attn(dev_bf16(np.concatenate(q)), dev_bf16(np.concatenate(k)), dev_bf16(np.concatenate(v)), 0.125,
                        cu_q=cu(q_lens), cu_kv=cu(lens), max_q_len=3, max_kv_len=1500)
    torch.cuda.synchronize()
    o = 0
    for i, m in enumerate(q_lens):
        assert_attn_close(out[o:o + m], oracle.decode_attn(q[i], k[i], v[i], 0.125)[0], f"request {i}")
        o += m


@pytest.mark.parametrize("lens,hq,hkv,d", [
    ([1281, 40], 12, 6, 64), ([1024, 1025, 3], 10, 5, 64), ([1281] * 3, 12, 6, 64),       # more than 16 heads: five chunks
    ([1300, 70, 900], 8, 4, 64), ([1281] + [33 + i for i in range(31)], 4, 2, 64),         # every CU, two heads: five chunks
    ([769, 5], 16, 8, 128), ([770, 300, 129, 768], 10, 5, 128), ([769, 100, 200], 10, 5, 128),
    ([1000] + [40 + 9 * i for i in range(31)], 4, 1, 128),
])
def test_ragged_batch_at_the_last_chunk_count(B, lens, hq, hkv, d):
    ragged_case(B, lens, [1] * len(lens), hq, hkv, d)


@pytest.mark.parametrize("kv_len,hq,hkv,d", [
    (1280, 6, 3, 64), (1281, 6, 3, 64), (1024, 20, 10, 64), (1025, 20, 10, 64), (768, 32, 16, 128), (769, 32, 16, 128), (769, 16, 8, 128),
])
def test_heads_that_do_not_divide_the_xcds(B, kv_len, hq, hkv, d):
    test_edges_match_oracle(B, 2, kv_len, hq, hkv, d, 0)


@pytest.mark.parametrize("n_nodes,kv_len,hq,hkv,d", [(26, 300, 8, 1, 128), (64, 700, 4, 2, 64), (40, 40, 4, 1, 64)])
def test_tree_over_a_short_cache(B, n_nodes, kv_len, hq, hkv, d):
    parent = synth.make_tree(n_nodes, 90 + n_nodes)
    masks = synth.ancestor_masks(parent)
    q, k, v = rnd_bits((n_nodes, hq, d), 5900), rnd_bits((kv_len, hkv, d), 5901), rnd_bits((kv_len, hkv, d), 5902)
    want, _ = oracle.tree_attn(q, k, v, masks, 0.1)
    out = B.tree_attn(dev_bf16(q), dev_bf16(k), dev_bf16(v), 0.1, torch.from_numpy(masks.view(np.int64)).cuda())
    torch.cuda.synchronize()
    assert_attn_close(out, want, f"tree {n_nodes} over {kv_len}")


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d", [
    (1, 1345, 14, 2, 64), (2, 1376, 14, 2, 64), (3, 1377, 4, 1, 64), (1, 961, 4, 1, 64),      # a last wave of 1, 32, 33, 1 keys
    (1, 897, 8, 2, 128), (6, 929, 16, 2, 128), (2, 769, 8, 1, 128), (8, 513, 32, 4, 128),
    (40, 1346, 4, 1, 64), (40, 898, 4, 1, 128),          # a block that lies across waves: the last one has 1 or 2 of its keys
])
def test_a_last_wave_of_few_keys(B, q_len, kv_len, hq, hkv, d):
    test_edges_match_oracle(B, q_len, kv_len, hq, hkv, d, 0)


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d,splits", [
    (1, 16257, 4, 1, 64, 128), (2, 2080, 8, 2, 64, 17),       # 128 keys a split and a last one of 1; 123 and 112
    (1, 2081, 4, 1, 64, 17), (4, 2049, 4, 4, 64, 16),         # 123 and 113; 129: one key too many for the four waves
    (1, 16384, 8, 8, 64, 128), (1, 16256, 8, 8, 64, 127),     # a head per XCD: the ring kernel from 128 splits on
])
def test_short_splits(B, q_len, kv_len, hq, hkv, d, splits):
    test_edges_match_oracle(B, q_len, kv_len, hq, hkv, d, splits)


def test_ragged_batch_of_short_splits(B):
    """128 keys a split; last splits of 1, 32, 33 and 128 keys, requests with fewer live splits than the launch, waves without keys."""
    ragged_case(B, [1280, 129, 160, 161, 3, 1024], [2, 1, 2, 1, 2, 2], 14, 2, 64, num_splits=10)


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d,splits", [(2, 1345, 14, 2, 64, 0), (6, 1000, 64, 8, 128, 0), (1, 1000, 12, 3, 64, 0),
                                                          (1, 2080, 14, 2, 64, 17)])
def test_head_major_caches(B, q_len, kv_len, hq, hkv, d, splits):
    q, k, v = (rnd_bits((n, h, d), 7200 + kv_len + i) for i, (n, h) in enumerate(((q_len, hq), (kv_len, hkv), (kv_len, hkv))))
    want, want_lse = oracle.decode_attn(q, k, v, 0.11)
    kd, vd = (dev_bf16(x).permute(1, 0, 2).contiguous().permute(1, 0, 2) for x in (k, v))
    out, lse = B.decode_attn(dev_bf16(q), kd, vd, 0.11, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    assert_attn_close(out, want, f"head-major q{q_len} kv{kv_len} {hq}/{hkv} d{d}")
    np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4)


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d,splits", [(6, 1000, 16, 2, 128, 0), (1, 1500, 14, 2, 64, 0), (2, 2080, 8, 2, 64, 17)])
@pytest.mark.parametrize("bumps", [((3, 120.0),), ((700, 60.0),), ((40, 60.0), (500, 150.0), (930, 40.0))])
def test_dominant_keys(B, q_len, kv_len, hq, hkv, d, splits, bumps):
    """Keys whose logits tower over the others by 2^40 .. 2^150: each wave has its own maximum, and the waves' parts meet."""
    scale, r = 0.088, np.random.default_rng(7300 + kv_len + int(bumps[0][1]))
    base = r.standard_normal(d).astype(np.float32)
    q = synth.f32_to_bf16_bits(base[None, None, :] + 0.3 * r.standard_normal((q_len, hq, d)).astype(np.float32))
    k = 0.2 * r.standard_normal((kv_len, hkv, d)).astype(np.float32)
    for pos, log2_units in bumps:
        k[pos] = (log2_units / (scale * np.log2(np.e) * float(base @ base))) * base[None, :]
    k, v = synth.f32_to_bf16_bits(k), rnd_bits((kv_len, hkv, d), 7301)
    want, want_lse = oracle.decode_attn(q, k, v, scale)
    out, lse = B.decode_attn(dev_bf16(q), dev_bf16(k), dev_bf16(v), scale, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    assert_attn_close(out, want, f"bumps {bumps} kv{kv_len}")
    np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4)


def test_balanced_pieces_of_few_tiles(B):
    """Fewer tiles than workgroups, one request just too long for the launch without splits."""
    ragged_case(B, [70, 5, 1100], [3, 3, 3], 8, 2, 128)
    ragged_case(B, [1537, 90], [1, 2], 14, 2, 64)
