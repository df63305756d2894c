"""GPU parity of specvlm_accept at the sizes where its kernels change what they do: as many rows as there
can be (129 with 31 and 32 chunks, more rows than one round of the merge takes), more chunks than a workgroup has threads, more
rows and chunks than one round of the argmax merge takes.  Bounds: those of the acceptance tests (greedy bit-exact,
sampling equal outside a margin of 1e-4)."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_accept as base
import test_gpu_tree as tree

pytestmark = pytest.mark.gpu
B = base.B


@pytest.mark.parametrize("batch,gamma,vocab,temp", [
    (1, 64, 253952, 1.0), (1, 64, 253953, 1.0), (1, 1, 8388609, 1.0), (2, 1, 8192, 0.9), (2, 2, 8193, 1.0),
])
def test_sampling(B, batch, gamma, vocab, temp):
    base.test_sampling_matches_oracle_outside_margin(B, batch, gamma, vocab, temp)


@pytest.mark.parametrize("batch,gamma,vocab,sigma", [(2, 15, 524288, 0.3), (1, 16, 532481, 0.3), (3, 33, 8193, 0.1)])
def test_greedy(B, batch, gamma, vocab, sigma):
    base.test_greedy_bit_exact(B, batch, gamma, vocab, sigma)


# short chunks (every wave has one step of 64 tokens up to 1024, two from 1025), eight chunks and nine (one and two groups of the merge)
@pytest.mark.parametrize("batch,gamma,vocab,temp", [
    (8, 3, 63, 1.0), (8, 3, 1024, 1.0), (8, 3, 1025, 1.0), (4, 2, 8192 + 1024, 0.8), (4, 2, 8192 + 1, 1.0), (2, 5, 65536, 1.0), (2, 5, 65537, 1.0),
])
def test_sampling_at_the_ends_of_chunks(B, batch, gamma, vocab, temp):
    base.test_sampling_matches_oracle_outside_margin(B, batch, gamma, vocab, temp)


# where the merge goes from one lane a row to 16 and back: 8 and 9 chunks, 16 and 17 rows, 65 rows of 15 to 49 chunks
@pytest.mark.parametrize("batch,gamma,vocab", [(2, 15, 65536), (2, 15, 65537), (2, 16, 65537), (1, 64, 122880),
                                               (1, 64, 401408), (3, 0, 70000)])
def test_greedy_at_the_merge_s_edges(B, batch, gamma, vocab):
    base.test_greedy_bit_exact(B, batch, gamma, vocab, 0.3)


@pytest.mark.parametrize("batch,n_nodes,vocab", [(4, 16, 65537), (4, 17, 65537), (4, 64, 65537), (4, 33, 140000)])
def test_tree_at_the_merge_s_edges(B, batch, n_nodes, vocab):
    tree.test_accept_tree_bit_exact_on_random_trees(B, batch, n_nodes, vocab)


def nan_rows():
    """Logits with NaN where a merge could keep one: at the first token of a chunk, of a thread's and of a wave's share,
    at token 0 (which then wins: nothing is greater), everywhere but in one place, and strewn about."""
    r = np.random.default_rng(77)
    x = r.standard_normal((8, 40000)).astype(np.float32)
    x[0, 8192], x[0, 25000] = np.nan, 9.0
    x[1, 0], x[1, 30000] = np.nan, 9.0
    x[2, :39999] = np.nan
    x[2, 0] = -np.inf
    x[3, ::8192], x[3, 9], x[3, 8192] = np.nan, 9.0, np.nan
    x[3, 0] = 0.0
    x[4, r.random(40000) < 0.3] = np.nan
    x[5, 64:8192:64], x[5, 8192 + 64], x[5, 64 + 256] = np.nan, np.nan, 9.0
    x[6, :] = np.nan
    x[7, 16384:], x[7, 0] = np.nan, -1.0
    return x


def test_a_nan_logit_is_never_the_largest(B):
    x = nan_rows()
    tokens = np.array([oracle.accept_greedy(row[None], np.zeros(0, np.int32))[1][0] for row in x], np.int32)
    n, out = B.accept(base.cuda(x[None]), base.cuda(tokens[None, :7]))
    parent = np.arange(-1, 7, dtype=np.int32)                          # a tree of one path drafts the same tokens
    nodes = np.concatenate([[0], tokens[:7]]).astype(np.int32)
    tn, _, tout = B.accept_tree(base.cuda(x[None]), base.cuda(nodes[None]), base.cuda(parent))
    torch.cuda.synchronize()
    assert out[0].cpu().tolist() == tokens.tolist() and n.item() == 7
    assert tout[0].cpu().tolist() == tokens.tolist() and tn.item() == 7


@pytest.mark.parametrize("vocab", [700, 8192, 20000])
def test_a_final_uniform_outside_its_range_stays_inside_the_row(B, vocab):
    """Outside [0, 1) nothing is promised but a token of the row; at 1 and above it is the last one with mass."""
    r = np.random.default_rng(vocab)
    x = r.standard_normal((5, 1, vocab)).astype(np.float32)
    x[:, 0, vocab - 40:] = -np.inf
    u = np.array([[-0.25], [-np.inf], [np.nan], [1.0], [2.0]], np.float32)
    n, out = B.accept(base.cuda(x), base.cuda(np.zeros((5, 0), np.int32)), uniforms=base.cuda(u))
    torch.cuda.synchronize()
    out = out.cpu().numpy().ravel()
    assert n.cpu().tolist() == [0] * 5
    assert ((0 <= out) & (out < vocab)).all() and out[3] == out[4] == vocab - 41
