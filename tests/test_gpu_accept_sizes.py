"""GPU parity of specvlm_accept at the sizes where its kernels change what they do: pass-1 partials of a request that just
fit the staging area and that do not (129 rows x 31 / 32 chunks), more chunks than the final kernel has threads, more
rows and chunks than one round of the argmax merge takes.  Bounds: those of the acceptance tests (greedy bit-exact,
sampling equal outside a margin of 1e-4)."""
import pytest

import test_gpu_accept as base

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
