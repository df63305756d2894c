"""GPU parity: specvlm_decode_attn (through the C ABI) against the fp64 oracle,
element by element, on seeded inputs spanning several tiles, splits and ragged
tails; tolerance max-abs 2e-2 / mean-abs 2e-3 (bf16 in, fp32 accumulate)."""
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


def run_case(B, q_len, kv_len, hq, hkv, d, seed, num_splits=0, scale=None, head_major=False,
             check_lse=True):
    scale = scale if scale is not None else 1.0 / np.sqrt(d)
    q, k, v = rnd_bits((q_len, hq, d), seed), rnd_bits((kv_len, hkv, d), seed + 1), rnd_bits((kv_len, hkv, d), seed + 2)
    want, want_lse = oracle.decode_attn(q, k, v, scale)
    qd, kd, vd = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    if head_major:      # [heads, tokens, d] storage viewed as [tokens, heads, d]
        kd = kd.permute(1, 0, 2).contiguous().permute(1, 0, 2)
        vd = vd.permute(1, 0, 2).contiguous().permute(1, 0, 2)
    out, lse = B.decode_attn(qd, kd, vd, scale, want_lse=True, num_splits=num_splits)
    torch.cuda.synchronize()
    tag = f"q{q_len} kv{kv_len} h{hq}/{hkv} d{d} splits{num_splits}"
    assert_attn_close(out, want, tag)
    if check_lse:
        np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4, err_msg=tag)
    return out


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d,splits", [
    (1, 1, 4, 1, 64, 0),           # a single key
    (1, 31, 4, 1, 64, 0),          # less than one tile
    (1, 32, 7, 1, 64, 1),
    (5, 1637, 4, 1, 64, 0),        # Tiny workload: gamma 4 over 1568 video + 64 text + block
    (5, 1637, 4, 1, 64, 1),
    (5, 1637, 4, 1, 64, 7),
    (1, 1511, 14, 2, 64, 0),       # draft-shaped decode over a pruned cache
    (6, 3000, 16, 2, 128, 0),      # 48 rows per kv head, 3 row blocks
    (6, 3000, 16, 2, 128, 5),
    (6, 1000, 16, 2, 128, 1),
    (8, 2077, 10, 2, 128, 3),      # group 5 (32B-shaped), gamma 7
    (8, 777, 16, 2, 128, 2),       # 64 rows: 4 row blocks
    (6, 2900, 28, 4, 128, 0),      # 7B-shaped heads (group 7): 42 rows, 3 row blocks with a ragged last one
    (1, 2900, 28, 4, 128, 0),
    (4, 515, 40, 8, 128, 0),
    (6, 6, 8, 1, 128, 0),          # cache holds only the block itself
    (3, 130, 2, 2, 64, 0),         # group 1
    (6, 9000, 8, 1, 128, 70),      # more splits than the merge kernel prefetches (12 groups x 3 = 36)
    (2, 9000, 4, 1, 64, 70),       # the same for d 64
    (6, 200, 8, 1, 128, 1),        # one split of three tiles and a bit: the ring wraps once
    (6, 70, 16, 2, 128, 0),        # a split shorter than the ring: its last tile is loaded twice
    (9, 900, 8, 1, 64, 0),         # 72 rows per kv head: two groups of three row blocks
    (16, 3000, 16, 2, 128, 0),     # chain of gamma 15 at group 8: 128 rows, two groups of four row blocks
    (16, 3000, 16, 2, 128, 1),
    (16, 700, 28, 4, 128, 3),      # group 7: 112 rows
    (64, 300, 16, 1, 64, 2),       # the longest block: 64 queries x group 16 = 1024 rows, sixteen groups
    (13, 13, 8, 1, 128, 0),        # more than 64 rows and nothing but the block itself
])
def test_matches_oracle(B, q_len, kv_len, hq, hkv, d, splits):
    run_case(B, q_len, kv_len, hq, hkv, d, seed=100 + q_len + kv_len, num_splits=splits)


@pytest.mark.parametrize("splits", [0, 1, 5])
@pytest.mark.parametrize("bumps", [((1000, 60.0),), ((1500, 150.0),), ((500, 60.0), (2000, 150.0), (2600, 40.0)),
                                   ((70, 120.0), (2990, 90.0))])
def test_dominant_keys_late_in_the_cache(B, splits, bumps):
    """Keys whose logits tower over everything before them (by 2^40 .. 2^150 in the softmax's own base-2
    units): away from the mask the kernel takes exponentials against the reference left by earlier
    chunks instead of tracking the maximum, and must fall back to the tracked form when a term no
    longer fits; either way the result is the oracle's."""
    from paper_2508_16201_amd.synth import f32_to_bf16_bits, bf16_bits_to_f32
    q_len, kv_len, hq, hkv, d, scale = 6, 3000, 16, 2, 128, 0.088
    rng = np.random.default_rng(4242 + len(bumps) + int(bumps[0][1]))
    base = rng.standard_normal(d).astype(np.float32)
    qf = base[None, None, :] + 0.3 * rng.standard_normal((q_len, hq, d)).astype(np.float32)   # rows nearly parallel
    kf = 0.2 * rng.standard_normal((kv_len, hkv, d)).astype(np.float32)
    vf = rng.standard_normal((kv_len, hkv, d)).astype(np.float32)
    unit = base / np.linalg.norm(base)
    for pos, log2_units in bumps:
        # logit (base-2 units) of a query row ~ scale * log2(e) * alpha * |base|
        alpha = log2_units / (scale * np.log2(np.e) * np.linalg.norm(base))
        kf[pos] = alpha * unit[None, :]
    q, k, v = f32_to_bf16_bits(qf), f32_to_bf16_bits(kf), f32_to_bf16_bits(vf)
    want, want_lse = oracle.decode_attn(q, k, v, scale)
    out, lse = B.decode_attn(dev_bf16(q), dev_bf16(k), dev_bf16(v), scale, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    tag = f"bumps {bumps} splits {splits}"
    assert_attn_close(out, want, tag)
    np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4, err_msg=tag)


def test_head_major_cache_layout(B):
    run_case(B, 6, 2500, 16, 2, 128, seed=7, head_major=True)
    run_case(B, 1, 900, 8, 2, 64, seed=8, head_major=True, num_splits=3)


def test_splits_agree_within_rounding(B):
    q, k, v = rnd_bits((6, 16, 128), 1), rnd_bits((4000, 2, 128), 2), rnd_bits((4000, 2, 128), 3)
    qd, kd, vd = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    a = B.decode_attn(qd, kd, vd, 0.088, num_splits=1).float()
    b = B.decode_attn(qd, kd, vd, 0.088, num_splits=9).float()
    torch.cuda.synchronize()
    # Two kernel results, no oracle here: one bf16 ulp of the output (2^-7 relative covers a step
    # across a binade), plus an absolute term for what does not scale with the output: the
    # probabilities are rounded to bf16 against each split's own running maximum, and the partial
    # outputs of the splits travel as bf16 (2^-9 of a partial that may be larger than the merged value
    # when values of both signs cancel).  Against the fp64 oracle either result is within 4e-4 here.
    tol = torch.maximum(a.abs(), b.abs()) * 2.0 ** -7 + 6e-4
    assert bool(((a - b).abs() <= tol).all())


def test_gamma_zero_equals_last_row_of_verify_block(B):
    # plain decode of the last block token == that token's row inside the verify call
    q, k, v = rnd_bits((6, 8, 128), 4), rnd_bits((1500, 1, 128), 5), rnd_bits((1500, 1, 128), 6)
    qd, kd, vd = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    block = B.decode_attn(qd, kd, vd, 0.09, num_splits=4)
    for t in (0, 3, 5):
        vis = 1500 - 6 + t + 1
        single = B.decode_attn(qd[t:t + 1], kd[:vis], vd[:vis], 0.09, num_splits=4)
        torch.cuda.synchronize()
        assert (block[t].float() - single[0].float()).abs().max().item() <= 4e-3


def test_large_logits_and_zero_scale(B):
    # peaked softmax (one dominant key) and the uniform limit
    run_case(B, 2, 700, 4, 1, 128, seed=9, scale=1.5)
    run_case(B, 2, 700, 4, 1, 128, seed=10, scale=0.0)


def test_ragged_batch_equals_per_request_calls(B):
    lens = [700, 33, 2049, 1280]
    q_lens = [6, 6, 1, 4]
    hq, hkv, d = 16, 2, 128
    qs = [rnd_bits((ql, hq, d), 20 + i) for i, ql in enumerate(q_lens)]
    ks = [rnd_bits((n, hkv, d), 30 + i) for i, n in enumerate(lens)]
    vs = [rnd_bits((n, hkv, d), 40 + i) for i, n in enumerate(lens)]
    cu_q = torch.tensor(np.concatenate([[0], np.cumsum(q_lens)]), dtype=torch.int32).cuda()
    cu_kv = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32).cuda()
    qd, kd, vd = dev_bf16(np.concatenate(qs)), dev_bf16(np.concatenate(ks)), dev_bf16(np.concatenate(vs))
    for splits in (0, 1, 6):
        out, lse = B.decode_attn(qd, kd, vd, 0.088, cu_q=cu_q, cu_kv=cu_kv, max_q_len=6,
                                 max_kv_len=max(lens), want_lse=True, num_splits=splits)
        torch.cuda.synchronize()
        o = 0
        for i in range(len(lens)):
            want, want_lse = oracle.decode_attn(qs[i], ks[i], vs[i], 0.088)
            assert_attn_close(out[o:o + q_lens[i]], want, f"req{i} splits{splits}")
            np.testing.assert_allclose(host_f64(lse[o:o + q_lens[i]]), want_lse, atol=2e-3, rtol=1e-4)
            o += q_lens[i]


@pytest.mark.parametrize("w", [synth.TINY, synth.V72B_1L])
def test_workload_verify_and_draft_shapes(B, w):
    t = synth.make_layer(w)
    scale = w.softmax_scale
    want, _ = oracle.decode_attn(t["q_block"], t["k"], t["v"], scale)
    out = B.decode_attn(dev_bf16(t["q_block"]), dev_bf16(t["k"]), dev_bf16(t["v"]), scale)
    torch.cuda.synchronize()
    assert_attn_close(out, want, w.name)


def test_full_size_72b_layer_sampled_rows(B):
    """configs[2] shape (12 806 keys, 64/8 heads, d 128, gamma 5) in the launch
    configuration the benchmark times; the oracle checks every row of every kv-head
    group (it computes rows one by one)."""
    w = synth.V72B_FULL
    t = synth.make_layer(w)
    scale = w.softmax_scale
    out, lse = B.decode_attn(dev_bf16(t["q_block"]), dev_bf16(t["k"]), dev_bf16(t["v"]), scale, want_lse=True)
    torch.cuda.synchronize()
    for g in range(w.n_kv_heads):
        hs = slice(g * 8, g * 8 + 8)
        want, want_lse = oracle.decode_attn(t["q_block"][:, hs], t["k"][:, g:g + 1], t["v"][:, g:g + 1], scale)
        assert_attn_close(out[:, hs], want, f"72b-full kv head {g}")
        np.testing.assert_allclose(host_f64(lse[:, hs]), want_lse, atol=2e-3, rtol=1e-4)


def test_argument_errors(B):
    q = torch.zeros((2, 4, 64), dtype=torch.bfloat16, device="cuda")
    k = torch.zeros((1, 1, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.SpecVLMError) as e:
        B.decode_attn(q, k, k, 0.1)                       # q_len > kv_len
    assert e.value.status == -1
    k3 = torch.zeros((8, 3, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.SpecVLMError):
        B.decode_attn(q, k3, k3, 0.1)                     # 4 % 3 != 0
    q96 = torch.zeros((1, 4, 96), dtype=torch.bfloat16, device="cuda")
    k96 = torch.zeros((8, 1, 96), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.SpecVLMError) as e:
        B.decode_attn(q96, k96, k96, 0.1)
    assert e.value.status == -2
    qbig = torch.zeros((65, 8, 64), dtype=torch.bfloat16, device="cuda")  # more than 64 queries per request
    kbig = torch.zeros((128, 1, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.SpecVLMError) as e:
        B.decode_attn(qbig, kbig, kbig, 0.1)
    assert e.value.status == -2
    # workspace too small
    qq = torch.zeros((1, 4, 64), dtype=torch.bfloat16, device="cuda")
    kk = torch.zeros((4096, 1, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.SpecVLMError) as e:
        B.decode_attn(qq, kk, kk, 0.1, num_splits=8, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -3


def test_full_size_32b_long_layer_sampled_rows(B):
    """configs[3] shape: 32 768 video + 256 text keys, 40/8 heads (group 5), d 128,
    gamma in {3, 5, 7}; the oracle checks every row of one kv-head group."""
    for gamma, g in ((3, 1), (5, 4), (7, 7)):
        w = synth.scaled(synth.V32B_LONG, gamma=gamma)
        t = synth.make_layer(w, layer=gamma)
        scale = w.softmax_scale
        out, lse = B.decode_attn(dev_bf16(t["q_block"]), dev_bf16(t["k"]), dev_bf16(t["v"]), scale, want_lse=True)
        torch.cuda.synchronize()
        hs = slice(g * 5, g * 5 + 5)
        want, want_lse = oracle.decode_attn(t["q_block"][:, hs], t["k"][:, g:g + 1], t["v"][:, g:g + 1], scale)
        assert_attn_close(out[:, hs], want, f"32b-long gamma {gamma} kv head {g}")
        np.testing.assert_allclose(host_f64(lse[:, hs]), want_lse, atol=2e-3, rtol=1e-4)


def test_ragged_batch_of_eight_in_one_launch(B):
    """configs[4]: 8 requests, video lengths 21..167 frames x 196 tokens + 256 text
    + the verify block, 64/8 heads, d 128, gamma 5, one launch with cu arrays.
    The oracle checks every request: all rows of one kv-head group each (the group
    changes with the request, so every head group is covered), and a second group
    of the shortest, the longest and one middle request."""
    frames = synth.ragged_frames()
    hq, hkv, d, g1 = 64, 8, 128, 6
    lens = [int(f) * 196 + 256 + g1 for f in frames]
    qs = [rnd_bits((g1, hq, d), 500 + i) for i in range(8)]
    ks = [rnd_bits((n, hkv, d), 600 + i) for i, n in enumerate(lens)]
    vs = [rnd_bits((n, hkv, d), 700 + i) for i, n in enumerate(lens)]
    cu_q = torch.tensor(np.arange(9) * g1, dtype=torch.int32).cuda()
    cu_kv = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32).cuda()
    qd, kd, vd = dev_bf16(np.concatenate(qs)), dev_bf16(np.concatenate(ks)), dev_bf16(np.concatenate(vs))
    scale = 1 / np.sqrt(d)
    out, lse = B.decode_attn(qd, kd, vd, scale, cu_q=cu_q, cu_kv=cu_kv, max_q_len=g1, max_kv_len=max(lens),
                             want_lse=True)
    torch.cuda.synchronize()
    order = np.argsort(lens)
    extra = {int(order[0]), int(order[4]), int(order[-1])}
    for i in range(8):
        for g in ([(3 * i + 1) % 8] + ([(3 * i + 5) % 8] if i in extra else [])):
            hs = slice(g * 8, g * 8 + 8)
            want, want_lse = oracle.decode_attn(qs[i][:, hs], ks[i][:, g:g + 1], vs[i][:, g:g + 1], scale)
            assert_attn_close(out[i * g1:(i + 1) * g1, hs], want, f"ragged request {i} kv head {g}")
            np.testing.assert_allclose(host_f64(lse[i * g1:(i + 1) * g1, hs]), want_lse, atol=2e-3, rtol=1e-4)


def _batch_case(B, lens, q_lens, hq, hkv, d, seed, scale=0.09):
    qs = [rnd_bits((ql, hq, d), seed + i) for i, ql in enumerate(q_lens)]
    ks = [rnd_bits((n, hkv, d), seed + 1000 + i) for i, n in enumerate(lens)]
    vs = [rnd_bits((n, hkv, d), seed + 2000 + i) for i, n in enumerate(lens)]
    cu_q = torch.tensor(np.concatenate([[0], np.cumsum(q_lens)]), dtype=torch.int32).cuda()
    cu_kv = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32).cuda()
    qd, kd, vd = dev_bf16(np.concatenate(qs)), dev_bf16(np.concatenate(ks)), dev_bf16(np.concatenate(vs))
    out, lse = B.decode_attn(qd, kd, vd, scale, cu_q=cu_q, cu_kv=cu_kv, max_q_len=max(q_lens),
                             max_kv_len=max(lens), want_lse=True)
    torch.cuda.synchronize()
    o = 0
    for i, ql in enumerate(q_lens):
        if ql:
            want, want_lse = oracle.decode_attn(qs[i], ks[i], vs[i], scale)
            assert_attn_close(out[o:o + ql], want, f"request {i} of lens {lens[:6]}...")
            np.testing.assert_allclose(host_f64(lse[o:o + ql]), want_lse, atol=2e-3, rtol=1e-4)
        o += ql


@pytest.mark.parametrize("lens,q_lens,hq,hkv,d", [
    # short requests: one launch without pieces
    ([70, 5, 129], [3, 3, 3], 8, 2, 128),
    # a request without queries in the middle, one key only, one long request that spans many workgroups
    ([300, 64, 1, 9000, 17], [6, 0, 1, 6, 2], 16, 2, 128),
    # one query per request (the single-row-block launch shape, tiles of 128 keys), head size 64
    ([513, 128, 2047, 31, 1024, 77], [1, 1, 1, 1, 1, 1], 14, 2, 64),
    # 64 requests: the largest batch that is cut into balanced pieces
    ([37 + 61 * i for i in range(64)], [1 + i % 3 for i in range(64)], 8, 1, 128),
    # the draft of the ragged configuration: 8 requests, one query each, 28/4 heads d 128, pruned caches
    ([int(f * 19.6) + 256 + 1 for f in (21, 63, 88, 101, 124, 133, 156, 167)], [1] * 8, 28, 4, 128),
    # 65 requests: uniform splits
    ([50 + 13 * i for i in range(65)], [2] * 65, 4, 1, 64),
])
def test_batches_with_library_chosen_pieces(B, lens, q_lens, hq, hkv, d):
    _batch_case(B, lens, q_lens, hq, hkv, d, seed=9000 + len(lens))
