"""GPU parity of specvlm_select and specvlm_top_p_count at the edges of what their kernels assume: tokens that fill the
threads' runs exactly, by one less and one more, the first and last size of every kernel (4, 16, 32 and 64 tokens a
thread), k and budget at both ends, keys that all coincide in one digit or in all, and a selection that reaches the NaN
keys, which the slots past the last token share;  batches of as many requests as there are CUs and one more, from where two share a
CU.  Exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2508_16201_amd import binding
    binding.lib()
    return binding


def i32(x):
    return torch.tensor([x], dtype=torch.int32).cuda()


def scores(kind, n, seed):
    r = np.random.default_rng(seed)
    s = np.exp(r.standard_normal(n)).astype(np.float32)
    if kind == "equal":
        s[:] = 0.25
    elif kind == "tight":                      # three equal leading digits
        s = (1.0 + 1e-5 * r.standard_normal(n)).astype(np.float32)
    elif kind == "nan":                        # fewer numbers than are taken
        s[r.random(n) < 0.9] = np.nan
        s[r.random(n) < 0.05] = -0.0
    return s


SIZES = [1, 2, 63, 1023, 1024, 1025, 4095, 4096, 4097, 12544, 16383, 16384, 16385, 32768, 32769, 65535, 65536]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kind", ["spread", "equal", "tight", "nan"])
def test_select(B, n, kind):
    s = scores(kind, n, n)
    dev = torch.from_numpy(s).cuda()
    for k, budget in {(0, n), (0, 1), (1, 1), (n, n), (n - 1, n), (n // 20, n // 10), (n // 2, n // 2 + n // 3), (n // 5, n)}:
        if not 0 <= k <= budget <= n or budget == 0:
            continue
        want, want_flags = oracle.select(s, k, budget)
        keep, flags = B.select(dev, i32(k), i32(budget), budget)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(keep.cpu().numpy(), want, err_msg=f"n {n} k {k} budget {budget} {kind}")
        np.testing.assert_array_equal(flags.cpu().numpy(), want_flags)


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("kind", ["spread", "equal", "nan"])
def test_top_p_count(B, n, kind):
    s = scores(kind, n, n + 1)
    dev = torch.from_numpy(s).cuda()
    for lam in (0.0, 0.25, 0.4, 1.0):
        lam = float(np.float32(lam))
        got = B.top_p_count(dev, lam).item()
        want, margin = oracle.top_p_count(s, lam, want_margin=True)
        if margin > 1e-6 or lam == 1.0:
            assert got == want, (n, kind, lam)


# keys that part in one digit of the descent (11, 11 and 10 bits) alone, its lowest and highest values among them, negative
# scores included: the thread that owns a digit, and the digits on both sides of a thread's and of a wave's share
@pytest.mark.parametrize("n", [2048, 4097, 16385, 32769, 65536])
@pytest.mark.parametrize("shift,bits", [(21, 11), (10, 11), (0, 10)])
def test_select_one_digit(B, n, shift, bits):
    r = np.random.default_rng(n + shift)
    digit = r.permutation(np.arange(n) % (1 << bits)).astype(np.uint32)
    key = (np.uint32(0xBF812345) & ~np.uint32(((1 << bits) - 1) << shift)) | (digit << np.uint32(shift))
    s = np.where(key >> 31 != 0, key & np.uint32(0x7FFFFFFF), ~key).astype(np.uint32).view(np.float32)
    dev = torch.from_numpy(s).cuda()
    for k in (1, n >> bits, (n >> bits) + 1, n // 16, n // 2 + 1, n - 1, n):
        want, want_flags = oracle.select(s, k, n)
        keep, flags = B.select(dev, i32(k), i32(n), n)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(keep.cpu().numpy(), want, err_msg=f"n {n} k {k} digit at {shift}")
        np.testing.assert_array_equal(flags.cpu().numpy(), want_flags, err_msg=f"n {n} k {k} digit at {shift}")


@pytest.mark.parametrize("batch,n", [(256, 1025), (257, 4), (257, 1025), (257, 4096), (300, 4097), (257, 16384), (257, 16385), (260, 32768), (257, 32769)])
def test_select_of_many_requests(B, batch, n):
    r = np.random.default_rng(batch + n)
    lens = np.minimum(r.integers(1, n + 1, batch) + np.where(r.random(batch) < 0.2, n, 0), n)
    lens[0] = n
    parts = [scores(("spread", "equal", "tight", "nan")[b % 4], v, b) for b, v in enumerate(lens)]
    budget = np.array([r.integers(0, v + 1) for v in lens], np.int32)
    k = np.array([r.integers(0, x + 1) for x in budget], np.int32)
    cu = [torch.from_numpy(np.concatenate([[0], np.cumsum(x)]).astype(np.int32)).cuda() for x in (lens, budget)]
    keep, flags = B.select(torch.from_numpy(np.concatenate(parts)).cuda(), torch.from_numpy(k).cuda(), torch.from_numpy(budget).cuda(),
                           int(budget.sum()), cu_video=cu[0], cu_keep=cu[1], max_n_video=n)
    torch.cuda.synchronize()
    want = [oracle.select(s, int(a), int(c)) for s, a, c in zip(parts, k, budget)]
    np.testing.assert_array_equal(keep.cpu().numpy(), np.concatenate([w[0] for w in want]))
    np.testing.assert_array_equal(flags.cpu().numpy(), np.concatenate([w[1] for w in want]))
