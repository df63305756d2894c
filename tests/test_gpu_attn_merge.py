"""GPU parity of the decode-attention merges where their launch changes: eight splits and nine, row counts on both sides of
the lines from which a group of threads takes a row, rows that do not fill the last workgroup, and ragged batches in which
requests have fewer live splits than the launch; partial results that 32-bit offsets do not reach.  Bounds: those of every
attention test."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev_bf16, host_f64, rnd_bits, assert_attn_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2508_16201_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d,splits", [
    (8, 1300, 32, 4, 128, 8), (8, 1300, 36, 4, 128, 8), (8, 1300, 36, 4, 128, 9),      # 256 and 288 rows: a workgroup each
    (11, 900, 24, 1, 64, 8), (11, 900, 24, 1, 64, 2),                                  # 264 rows
    (13, 300, 63, 3, 128, 3), (13, 1025, 63, 3, 128, 8),                               # 273 rows a head
])
def test_uniform_splits(B, q_len, kv_len, hq, hkv, d, splits):
    q, k, v = (rnd_bits((n, h, d), 6000 + kv_len + i) for i, (n, h) in enumerate(((q_len, hq), (kv_len, hkv), (kv_len, hkv))))
    scale = 1.0 / np.sqrt(d)
    want, want_lse = oracle.decode_attn(q, k, v, scale)
    out, lse = B.decode_attn(dev_bf16(q), dev_bf16(k), dev_bf16(v), scale, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    assert_attn_close(out, want, f"q{q_len} kv{kv_len} {hq}/{hkv} d{d} splits {splits}")
    np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4)


# twelve groups of threads: a thread's splits are three, four, eight, sixteen and 22 at most, by the launch
@pytest.mark.parametrize("splits", [36, 37, 48, 49, 96, 97, 192, 193, 255, 256])
@pytest.mark.parametrize("hq,hkv,d", [(4, 1, 64), (6, 2, 128)])
def test_uniform_splits_up_to_the_most(B, splits, hq, hkv, d):
    test_uniform_splits(B, 2, 128 * splits - 1, hq, hkv, d, splits)


def test_ragged_batch_with_named_splits(B):
    lens, q_lens, hq, hkv, d = [1500, 3, 257, 1024], [6, 3, 2, 6], 64, 4, 128
    q, k, v = [], [], []
    for i, (n, m) in enumerate(zip(lens, q_lens)):
        q.append(rnd_bits((m, hq, d), 6600 + i)); k.append(rnd_bits((n, hkv, d), 6700 + i)); v.append(rnd_bits((n, hkv, d), 6800 + i))
    cu = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32).cuda()  # noqa: E731
    out = B.decode_attn(dev_bf16(np.concatenate(q)), dev_bf16(np.concatenate(k)), dev_bf16(np.concatenate(v)), 0.088,
                        cu_q=cu(q_lens), cu_kv=cu(lens), max_q_len=6, max_kv_len=1500, num_splits=6)
    torch.cuda.synchronize()
    o = 0
    for i, m in enumerate(q_lens):
        assert_attn_close(out[o:o + m], oracle.decode_attn(q[i], k[i], v[i], 0.088)[0], f"request {i}")
        o += m


# live splits of a request: fewer than the groups, one more, a thread's first eight full, one more, all;  the last two heads make more than 512 workgroups
FEW_LIVE = [(4, 1, 64, 2), (6, 2, 128, 2), (32, 4, 64, 4), (32, 4, 128, 4)]


@pytest.mark.parametrize("splits", [40, 64, 100, 200])
@pytest.mark.parametrize("hq,hkv,d,q_len", FEW_LIVE)
def test_ragged_batch_of_few_live_splits(B, splits, hq, hkv, d, q_len):
    lens = [q_len, 11 * 128 - 5, 13 * 128, 128 * splits] + [n * 128 - 1 for n in (37, 49, 96, 97) if n < splits]
    q, k, v = [], [], []
    for i, n in enumerate(lens):
        q.append(rnd_bits((q_len, hq, d), 7300 + i)); k.append(rnd_bits((n, hkv, d), 7400 + i)); v.append(rnd_bits((n, hkv, d), 7500 + i))
    cu = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32).cuda()  # noqa: E731
    out, lse = B.decode_attn(dev_bf16(np.concatenate(q)), dev_bf16(np.concatenate(k)), dev_bf16(np.concatenate(v)), 0.1, cu_q=cu([q_len] * len(lens)),
                             cu_kv=cu(lens), max_q_len=q_len, max_kv_len=max(lens), num_splits=splits, want_lse=True)
    torch.cuda.synchronize()
    for i, n in enumerate(lens):
        want, want_lse = oracle.decode_attn(q[i], k[i], v[i], 0.1)
        assert_attn_close(out[i * q_len:(i + 1) * q_len], want, f"request {i} of {n} keys")
        np.testing.assert_allclose(host_f64(lse[i * q_len:(i + 1) * q_len]), want_lse, atol=2e-3, rtol=1e-4)


@pytest.mark.parametrize("q_len,kv_len,hq,hkv,d,splits", [
    (12, 700, 64, 8, 128, 4), (11, 700, 64, 8, 128, 4),                    # 768 and 704 rows, a head per XCD
    (24, 1025, 64, 8, 64, 8), (24, 1100, 64, 8, 64, 9), (23, 300, 64, 8, 64, 2),      # 1536 and 1472 at head size 64
    (28, 600, 64, 2, 128, 3), (27, 600, 64, 2, 128, 3), (56, 500, 64, 2, 64, 4),      # 1792, 1728 and 3584 rows, fewer heads
    (37, 400, 49, 7, 128, 2), (64, 300, 57, 3, 64, 2),                     # 1813 and 3648: rows that do not fill the last workgroup
])
def test_uniform_splits_of_many_rows(B, q_len, kv_len, hq, hkv, d, splits):
    test_uniform_splits(B, q_len, kv_len, hq, hkv, d, splits)


def test_ragged_batch_of_many_rows(B):
    lens, q_lens, hq, hkv, d = [900, 20, 257, 640], [9, 9, 2, 4], 64, 8, 128     # 2304 rows at most, 1 to 6 live splits
    q, k, v = [], [], []
    for i, (n, m) in enumerate(zip(lens, q_lens)):
        q.append(rnd_bits((m, hq, d), 6900 + i)); k.append(rnd_bits((n, hkv, d), 7000 + i)); v.append(rnd_bits((n, hkv, d), 7100 + i))
    cu = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32).cuda()  # noqa: E731
    out = B.decode_attn(dev_bf16(np.concatenate(q)), dev_bf16(np.concatenate(k)), dev_bf16(np.concatenate(v)), 0.088,
                        cu_q=cu(q_lens), cu_kv=cu(lens), max_q_len=9, max_kv_len=900, num_splits=6)
    torch.cuda.synchronize()
    o = 0
    for i, m in enumerate(q_lens):
        assert_attn_close(out[o:o + m], oracle.decode_attn(q[i], k[i], v[i], 0.088)[0], f"request {i}")
        o += m


def test_partials_beyond_32_bit_offsets(B):
    """480000 rows: the partial results of split 35 of 0 to 36, the last one that a workgroup requests together with the first,
    lie 4.3e9 bytes behind those, and its keys are the ones that every query looks at."""
    q_len, kv_len, hq, d, splits = 64, 37 * 128, 7500, 128, 37
    g = torch.Generator(device="cuda")
    g.manual_seed(66)
    at = torch.randn(d, generator=g, device="cuda")
    q = (at + 0.3 * torch.randn((q_len, hq, d), generator=g, device="cuda")).bfloat16()
    k = torch.randn((kv_len, 1, d), generator=g, device="cuda").bfloat16()
    v = torch.randn((kv_len, 1, d), generator=g, device="cuda").bfloat16()
    k[35 * 128:36 * 128] = (at + 0.5 * torch.randn((128, 1, d), generator=g, device="cuda")).bfloat16()
    scale = 1.0 / np.sqrt(d)
    out, lse = B.decode_attn(q, k, v, scale, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    rows = torch.randint(q_len * hq, (64,), generator=g, device="cuda")
    logits = (q.view(-1, d)[rows].double() @ k[:, 0].double().T) * scale
    hidden = torch.arange(kv_len, device="cuda")[None, :] > (kv_len - q_len + rows // hq)[:, None]
    logits.masked_fill_(hidden, float("-inf"))
    want = (logits.softmax(-1) @ v[:, 0].double()).cpu().numpy()
    assert np.abs(want).max() > 0.2
    assert_attn_close(out.view(-1, d)[rows], want, "sampled rows")
    np.testing.assert_allclose(host_f64(lse).reshape(-1)[rows.cpu().numpy()], logits.logsumexp(-1).cpu().numpy(), atol=2e-3, rtol=1e-4)
