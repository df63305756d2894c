"""GPU parity of the sampling acceptance whose last workgroup of a request finishes the call: 64 and 65 chunks (one and two
trips of a lane per chunk), final uniforms on both sides of every segment's and chunk's end, a workspace full of other
contents, and replays of a captured call with eager calls on the same workspace between them.  The bound of every sampling
test (equal outside a margin of 1e-4; test_gpu_accept_order.py has none); replays are equal bit for bit."""
import numpy as np
import pytest
import torch

import test_gpu_accept as base

pytestmark = pytest.mark.gpu
B = base.B


@pytest.mark.parametrize("batch,gamma,vocab,temp", [(1, 1, 524288, 1.0), (1, 1, 524289, 1.0), (9, 1, 16384, 1.0), (3, 64, 9000, 1.0)])
def test_sampling(B, batch, gamma, vocab, temp):
    base.test_sampling_matches_oracle_outside_margin(B, batch, gamma, vocab, temp)


@pytest.mark.parametrize("vocab", [1024, 8192, 8192 + 700, 40000])
def test_goals_around_the_ends_of_segments_and_chunks(B, vocab):
    """One row of equal logits: token v owns [v / vocab, (v + 1) / vocab), so a uniform in the middle of that interval
    names v whatever the rounding of 40000 fp32 sums (2^-24 * 40000 / 2 < 1e-2 of an interval's share of the total)."""
    ends = {vocab}
    for lo in range(0, vocab, 8192):                     # (a short chunk has narrower segments)
        size = min(vocab - lo, 8192)
        ends |= set(range(lo, lo + size, ((size + 15) // 16 + 63) & ~63))
    tokens = sorted({t for e in ends for t in (e - 1, e, e + 1) if 0 <= t < vocab})
    u = ((np.array(tokens, np.float64) + 0.5) / vocab).astype(np.float32)[:, None]
    x = np.zeros((len(tokens), 1, vocab), np.float32)
    n, out = B.accept(base.cuda(x), base.cuda(np.zeros((len(tokens), 0), np.int32)), uniforms=base.cuda(u))
    torch.cuda.synchronize()
    assert n.cpu().tolist() == [0] * len(tokens)
    assert out.cpu().numpy().ravel().tolist() == tokens


def test_replays_between_eager_calls_on_one_workspace(B):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    batch, gamma, vocab = 3, 4, 30000
    need = max(B.accept_workspace_bytes(b, gamma, vocab, True) for b in (1, batch))
    ws = torch.full((need,), 0xff, dtype=torch.uint8, device="cuda")

    def inputs(b):
        t = 2.0 * torch.randn((b, gamma + 1, vocab), generator=g, device="cuda")
        d = t[:, :gamma] + 0.5 * torch.randn((b, gamma, vocab), generator=g, device="cuda")
        return t, d.argmax(-1).to(torch.int32), d.contiguous(), torch.rand((b, gamma + 1), generator=g, device="cuda")

    def call(x, **kw):
        return B.accept(x[0], x[1], draft_logits=x[2], uniforms=x[3], **kw)

    mine, other = inputs(batch), inputs(1)
    want = [t.clone() for t in call(mine, workspace=torch.zeros(need, dtype=torch.uint8, device="cuda"))]
    n = torch.empty(batch, dtype=torch.int32, device="cuda")
    out = torch.empty((batch, gamma + 1), dtype=torch.int32, device="cuda")
    call(mine, workspace=ws, n_accepted=n, out_tokens=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(mine, workspace=ws, n_accepted=n, out_tokens=out)
    for _ in range(4):
        n.fill_(-7), out.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(n, want[0]) and torch.equal(out, want[1])
        call(other, workspace=ws)
        ws.fill_(0xff)
        torch.cuda.synchronize()


# last chunks of one token, one chunk that is not full, many requests and one alone
@pytest.mark.parametrize("batch,gamma,vocab", [(7, 2, 73728), (7, 2, 73729), (64, 1, 4097), (65, 1, 4097), (32, 1, 8193), (33, 1, 8193),
                                               (1, 3, 4096), (2, 3, 1025)])
def test_chunk_sizes(B, batch, gamma, vocab):
    base.test_sampling_matches_oracle_outside_margin(B, batch, gamma, vocab, 1.0)
