"""The sums of specvlm_accept's sampling mode in fp32 and in their order, in plain numpy.

The drawn token is where fp32 sums put the uniform, so a uniform within rounding of a step of the CDF is decided by the
order of the sums.  That order depends on the vocabulary alone:

  normaliser   per chunk of 8192 tokens: 256 running sums (token mod 256, ascending), each wave of 64 of them by
               lane ^ 32, 16, 8, 4, 2, 1, the four waves as (0 + 1) + (2 + 3);  chunks in ascending order, eight to a
               group, rescaled to the maximum so far at the start of a group
  chunk mass   the weights of a chunk, summed as above;  total and prefixes: running sums over the chunks
  segment      a sixteenth of a chunk, rounded up to 64 tokens: 64 running sums (token mod 64), then lane ^ 32 ... 1;
               prefixes: running sums over the segments, from the chunk's prefix
  token        64 tokens at a time: sums over the last 2, 4, 8, ... 64 tokens, each from two of the half length

Logits are integers and log2(e) / temperature is 1, so that every exponential is a power of two and all that rounds
is the additions and the divisions; a contracted multiply-add rounds no differently then.
"""
import numpy as np

F = np.float32
TEMPERATURE = float(F(1.4426950408889634))
CHUNK, SEGS = 8192, 16


def xor_tree(x):
    """The sum over lanes x[..., 64] as lane ^ 32, ^ 16, ... leave it in every lane."""
    for off in (32, 16, 8, 4, 2, 1):
        x = (x + x[..., np.arange(64) ^ off]).astype(F)
    return x[..., 0]


def running(x):
    """Running sums over the first axis, from 0."""
    s = np.zeros(x.shape[1:], F)
    for v in x:
        s = (s + v).astype(F)
    return s


def chunk_sums(w):
    """w [vocab] -> one sum per chunk."""
    n = (len(w) + CHUNK - 1) // CHUNK
    x = np.zeros(n * CHUNK, F)
    x[:len(w)] = w
    waves = xor_tree(running(x.reshape(n, CHUNK // 256, 256).transpose(1, 0, 2)).reshape(n, 4, 64))
    return ((waves[:, 0] + waves[:, 1]).astype(F) + (waves[:, 2] + waves[:, 3]).astype(F)).astype(F)


def normaliser(row):
    """(max, sum of powers of two) of a row of whole-numbered logits."""
    n = (len(row) + CHUNK - 1) // CHUNK
    tops = [row[c * CHUNK:(c + 1) * CHUNK].max() for c in range(n)]
    sums = chunk_sums(np.exp2(row - np.repeat(tops, CHUNK)[:len(row)]).astype(F))
    m, z = F(-np.inf), F(0)
    for c0 in range(0, n, 8):
        top = max([m, *tops[c0:c0 + 8]])
        z = F(z * np.exp2(F(m - top)))
        for c in range(c0, min(n, c0 + 8)):
            z = F(z + F(sums[c] * np.exp2(F(tops[c] - top))))
        m = top
    return m, z


class Drawn:
    """The CDF of one row (or of the residual of two): token(u) for a final uniform u, and its steps."""

    def __init__(self, target, draft=None):
        m, z = normaliser(target)
        w = (np.exp2(target - m).astype(F) * (F(1) / z)).astype(F)
        if draft is not None:
            m, z = normaliser(draft)
            w = np.maximum((w - (np.exp2(draft - m).astype(F) * (F(1) / z)).astype(F)).astype(F), F(0))
        self.w, self.mass = w, chunk_sums(w)
        self.before = np.concatenate([[F(0)], np.cumsum(self.mass, dtype=F)[:-1]])      # (numpy's cumsum is sequential)
        self.total = running(self.mass)

    def segments(self, chunk):
        lo, hi = chunk * CHUNK, min(len(self.w), (chunk + 1) * CHUNK)
        width = ((hi - lo + SEGS - 1) // SEGS + 63) // 64 * 64
        w = np.zeros(SEGS * width, F)
        w[:hi - lo] = self.w[lo:hi]
        w = w.reshape(SEGS, width // 64, 64)
        mass = xor_tree(running(w.transpose(1, 0, 2)))
        prefix = np.cumsum(np.concatenate([[self.before[chunk]], mass]), dtype=F)[:-1]
        return lo, width, w, mass, prefix

    def walk(self, w, prefix):
        """Cumulative mass behind every token of a segment w [steps, 64]."""
        incl = w.copy()
        for off in (1, 2, 4, 8, 16, 32):
            t = incl.copy()
            t[:, off:] = (incl[:, off:] + incl[:, :-off]).astype(F)
            incl = t
        c, cum = prefix, []
        for step in incl:
            cum.append((c + step).astype(F))
            c = F(c + step[63])
        return np.array(cum)

    def token(self, u):
        goal = F(F(u) * self.total)
        fits = np.flatnonzero((self.mass > 0) & (self.before <= goal))
        chunk = fits[-1] if len(fits) else 0
        lo, width, w, mass, prefix = self.segments(chunk)
        fits = np.flatnonzero((mass > 0) & (prefix <= goal))
        seg = fits[-1] if len(fits) else 0
        passed = np.flatnonzero((w[seg] > 0) & (self.walk(w[seg], prefix[seg]) > goal))
        massive = np.flatnonzero(w[seg] > 0)
        return int(lo + (seg * width + (passed[0] if len(passed) else massive[-1]) if len(massive) else 0))

    def steps(self, tokens):
        """The cumulative mass behind each of these tokens, as a share of the total."""
        out = []
        for t in tokens:
            lo, width, w, _, prefix = self.segments(t // CHUNK)
            seg, at = divmod(t - lo, width)
            out.append(float(self.walk(w[seg], prefix[seg]).ravel()[at]) / float(self.total))
        return np.array(out)


def probability(row, token):
    m, z = normaliser(row)
    return F(np.exp2(F(row[token] - m)) / z)


def accept(target, draft, tokens, uniforms):
    """(n accepted, output tokens) of one request."""
    gamma = len(tokens)
    n = 0
    while n < gamma and F(uniforms[n] * probability(draft[n], tokens[n])) < probability(target[n], tokens[n]):
        n += 1
    y = Drawn(target[n], draft[n] if n < gamma else None).token(uniforms[gamma])
    return n, [*tokens[:n], y] + [-1] * (gamma - n)
