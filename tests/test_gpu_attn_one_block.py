"""GPU parity of one block of query rows where its launch changes: splits of 127 and of 128 keys, and with fewer, as many
and more tiles than the ring is deep, of caches below the streamed size and above it; balanced pieces of it.  Bounds: those of
every attention test."""
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


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kv_len,splits", [(254, 2), (255, 2), (256, 2), (257, 2), (385, 2), (511, 2), (513, 2), (640, 2), (641, 2),
                                           (1283, 2), (128, 1), (129, 1), (1000, 1), (1537, 4)])
def test_splits_of_one_row_block(B, kv_len, splits, d):
    q_len, hq, hkv = 3, 10, 2                                     # 15 rows a kv head
    q, k, v = (rnd_bits((n, h, d), 9000 + kv_len + i) for i, (n, h) in enumerate(((q_len, hq), (kv_len, hkv), (kv_len, hkv))))
    scale = 1.0 / np.sqrt(d)
    want, want_lse = oracle.decode_attn(q, k, v, scale)
    out, lse = B.decode_attn(dev_bf16(q), dev_bf16(k), dev_bf16(v), scale, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    assert_attn_close(out, want, f"kv{kv_len} d{d} splits {splits}")
    np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4)


# (head size, kv heads, splits) with loader waves from 164 keys a split on: workgroups in one round, three of them to four CUs and one to each, and several
STREAMED = [(128, 64, 2), (64, 100, 2), (64, 128, 2), (64, 130, 4)]


@pytest.mark.parametrize("split_keys", [164, 192, 255, 257, 321, 641])            # 3 to 11 tiles, the last of 1 to 64 keys
@pytest.mark.parametrize("d,hkv,splits", STREAMED)
def test_splits_of_one_row_block_of_a_streamed_cache(B, d, hkv, splits, split_keys):
    q_len, hq, kv_len = 3, 2 * hkv, splits * split_keys
    q, k, v = (rnd_bits((n, h, d), 9700 + kv_len + i) for i, (n, h) in enumerate(((q_len, hq), (kv_len, hkv), (kv_len, hkv))))
    scale = 1.0 / np.sqrt(d)
    want, want_lse = oracle.decode_attn(q, k, v, scale)
    out, lse = B.decode_attn(dev_bf16(q), dev_bf16(k), dev_bf16(v), scale, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    assert_attn_close(out, want, f"{hkv} heads d{d} splits of {split_keys}")
    np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4)


# long splits of a cache below the streamed size, which size 128 has loader waves for, and eight heads whose keys lie side by side a head, which has size 64
# four ring stages for one block of rows and for two
@pytest.mark.parametrize("q_len,hq,hkv,d,splits,split_keys", [
    (1, 7, 1, 128, 3, 699), (1, 7, 1, 128, 3, 700), (3, 4, 1, 128, 2, 767), (2, 6, 3, 128, 2, 833), (2, 16, 8, 64, 3, 1400), (1, 16, 16, 64, 2, 1153), (20, 16, 8, 64, 4, 1100)])
def test_long_splits_of_heads_apart(B, q_len, hq, hkv, d, splits, split_keys):
    kv_len = splits * split_keys
    q, k, v = (rnd_bits((n, h, d), 9900 + kv_len + i) for i, (n, h) in enumerate(((q_len, hq), (kv_len, hkv), (kv_len, hkv))))
    apart = lambda x: dev_bf16(x).transpose(0, 1).contiguous().transpose(0, 1)  # noqa: E731
    scale = 1.0 / np.sqrt(d)
    want, want_lse = oracle.decode_attn(q, k, v, scale)
    out, lse = B.decode_attn(dev_bf16(q), apart(k), apart(v), scale, want_lse=True, num_splits=splits)
    torch.cuda.synchronize()
    assert_attn_close(out, want, f"{hkv} heads d{d} splits of {split_keys}")
    np.testing.assert_allclose(host_f64(lse), want_lse, atol=2e-3, rtol=1e-4)


@pytest.mark.parametrize("d", [64, 128])
def test_balanced_pieces_of_one_row_block(B, d):
    lens, hq, hkv = [3000, 1, 63, 65, 2049, 128], 32, 8
    q, k, v = [], [], []
    for i, n in enumerate(lens):
        q.append(rnd_bits((1, hq, d), 9400 + i)); k.append(rnd_bits((n, hkv, d), 9500 + i)); v.append(rnd_bits((n, hkv, d), 9600 + i))
    cu = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32).cuda()  # noqa: E731
    out = B.decode_attn(dev_bf16(np.concatenate(q)), dev_bf16(np.concatenate(k)), dev_bf16(np.concatenate(v)), 0.1,
                        cu_q=cu([1] * len(lens)), cu_kv=cu(lens), max_q_len=1, max_kv_len=3000)
    torch.cuda.synchronize()
    for i in range(len(lens)):
        assert_attn_close(out[i:i + 1], oracle.decode_attn(q[i], k[i], v[i], 0.1)[0], f"request {i}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lens,hq,hkv,pieces", [([2500, 2500], 28, 4, [20, 20]), ([1300, 1, 129], 40, 8, [11, 1, 2]), ([20000, 300], 12, 3, [84, 2])])
def test_balanced_pieces_are_of_128_keys_and_more(B, lens, hq, hkv, pieces, d):
    """Fewer units of 128 keys than groups of workgroups are a piece each; the last case has 160 for 85 groups."""
    cu = lambda x: torch.tensor(np.concatenate([[0], np.cumsum(x)]), dtype=torch.int32).cuda()  # noqa: E731
    n = len(lens)
    g = torch.Generator(device="cuda")
    g.manual_seed(97)
    k = torch.randn((sum(lens), hkv, d), generator=g, device="cuda").bfloat16()
    work = B.new_workspace(B.decode_attn_workspace_bytes(n, 1, max(lens), hq, hkv, d)).zero_()
    B.decode_attn(k[:n].repeat(1, hq // hkv, 1), k, k, 0.1, cu_q=cu([1] * n), cu_kv=cu(lens), max_q_len=1, max_kv_len=max(lens), workspace=work)
    slots = (256 + n * hkv) * 16                                       # partial outputs, maxima and sums, then the table of pieces
    at = (slots * d * 2 + 255) // 256 * 256 + (slots * 8 + 255) // 256 * 256
    table = work[at:at + n * hkv * 8].view(torch.int32).view(n, hkv, 2).cpu()
    assert table[:, :, 1].tolist() == [[x] * hkv for x in pieces]
