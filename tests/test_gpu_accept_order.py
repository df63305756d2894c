"""Sampling acceptance where rounding decides: final uniforms on the steps of the CDF and their fp32 neighbours, at the ends
of chunks and segments and in between, and acceptance tests at equality.  The token has to be the one that fp32 sums
in the documented order give (tests/sampling_order.py), exactly, and a request's tokens must not depend on the others in its
batch.  Inputs round in sums and divisions only, so nothing is allowed to differ."""
import numpy as np
import pytest
import torch

import sampling_order as order
import test_gpu_accept as base
from test_launches import least_bytes

pytestmark = pytest.mark.gpu
B = base.B
F = np.float32


def logits(r, *shape):
    """Whole numbers from -30 on: powers of two that no fp32 sum of thousands holds exactly."""
    return np.maximum(-r.geometric(0.15, shape), -30).astype(F)


def neighbours(u):
    u = np.asarray(u).astype(F)
    u = np.concatenate([np.nextafter(u, F(0)), u, np.nextafter(u, F(1))])
    return u[(u >= 0) & (u < 1)]


def call(B, target, draft, tokens, uniforms):
    n, out = B.accept(base.cuda(target), base.cuda(tokens), draft_logits=None if draft is None else base.cuda(draft),
                      uniforms=base.cuda(uniforms), temperature=order.TEMPERATURE)
    torch.cuda.synchronize()
    return n.cpu().numpy(), out.cpu().numpy()


# one short chunk and its ends, one chunk, a chunk and a bit, a last chunk whose segments are 64 wide, 19 chunks, one and two trips
# of the merge (32 and 33 chunks) and of the walk over the chunks (64 and 65)
@pytest.mark.parametrize("vocab", [63, 1000, 1024, 1025, 8192, 8193, 8892, 40000, 152064, 262144, 262145, 524288, 524289])
def test_final_uniforms_on_steps_of_the_cdf(B, vocab):
    r = np.random.default_rng(vocab)
    x = logits(r, vocab)
    cdf = order.Drawn(x)
    at = set(r.integers(0, vocab, 12).tolist())
    for chunk in {0, (vocab - 1) // order.CHUNK, int(r.integers((vocab - 1) // order.CHUNK + 1))}:
        lo, width, w, _, _ = cdf.segments(chunk)
        at |= {lo + seg * width + d for seg in r.permutation(order.SEGS)[:4].tolist() for d in (-1, 0)}
    at = [t for t in sorted(at) if 0 <= t < vocab]
    u = neighbours(cdf.steps(at))[:, None]
    target = np.broadcast_to(x, (len(u), 1, vocab))
    n, out = call(B, target, None, np.zeros((len(u), 0), np.int32), u)
    assert (n == 0).all()
    want = [cdf.token(v) for v in u.ravel()]
    assert out.ravel().tolist() == want, [(v, a, b) for v, a, b in zip(u.ravel(), out.ravel(), want) if a != b]


def requests(vocab, gamma, seed):
    """Requests that leave at every position: their tests at equality and next to it, their final uniform on a step."""
    r = np.random.default_rng(seed)
    target = logits(r, gamma + 1, vocab)
    draft = np.minimum(target[:gamma] + r.integers(-1, 2, (gamma, vocab)), 0).astype(F)
    tokens = r.integers(0, vocab, gamma).astype(np.int32)
    edge = np.array([order.probability(target[i], t) / order.probability(draft[i], t) for i, t in enumerate(tokens)], F)
    out = []
    for stop in range(gamma + 1):
        cdf = order.Drawn(target[stop], draft[stop] if stop < gamma else None)
        step = cdf.steps([r.choice(np.flatnonzero(cdf.w > 0))])
        for final in neighbours(step):
            u = np.minimum(np.nextafter(edge, F(0)), F(0.999))           # (just inside, or at equality from here on)
            if stop < gamma:
                u[stop] = F(0.99999994) if edge[stop] >= 1 else edge[stop]
            out.append(np.append(u, final).astype(F))
    return target, draft, tokens, np.array(out)


@pytest.mark.parametrize("vocab,gamma", [(700, 3), (1024, 2), (8192, 3), (30000, 4), (152064, 2)])
def test_tests_at_equality_and_alone_as_in_any_batch(B, vocab, gamma):
    target, draft, tokens, u = requests(vocab, gamma, vocab + gamma)
    want = [order.accept(target, draft, tokens, x) for x in u]

    def rows(count):
        pick = [i % len(u) for i in range(count)]
        n, out = call(B, *(np.broadcast_to(t, (count, *t.shape)) for t in (target, draft, tokens)), u[pick])
        for i, b in zip(pick, range(count)):
            assert (n[b], out[b].tolist()) == want[i], (count, b, n[b], out[b].tolist(), want[i])

    for i in range(len(u)):
        n, out = call(B, target[None], draft[None], tokens[None], u[i][None])
        assert (n[0], out[0].tolist()) == want[i], (i, n[0], out[0].tolist(), want[i])
    for count in (2, 4, 16, 70):
        rows(count)


@pytest.mark.parametrize("vocab,gamma,count", [(700, 3, 4), (8192, 3, 9), (30000, 4, 9), (30000, 4, 70), (530000, 1, 6)])
def test_workspace_without_the_segments_masses(B, vocab, gamma, count):
    target, draft, tokens, u = requests(vocab, gamma, vocab + 7)
    pick = [i % len(u) for i in range(count)]
    args = [base.cuda(np.broadcast_to(t, (count, *t.shape))) for t in (target, tokens, draft)] + [base.cuda(u[pick])]
    least = least_bytes(count, gamma, vocab)
    buf = torch.full((least + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    n, out = B.accept(args[0], args[1], draft_logits=args[2], uniforms=args[3], temperature=order.TEMPERATURE, workspace=buf[:least])
    torch.cuda.synchronize()
    assert (buf[least:] == 0x5a).all()
    want = [order.accept(target, draft, tokens, x) for x in u]
    for i, a, b in zip(pick, n.tolist(), out.tolist()):
        assert (a, b) == want[i], (i, a, b, want[i])
