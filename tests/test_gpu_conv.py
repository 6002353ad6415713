"""The int8 convolution kernels at the edges of their tiles and instance
groups, bit-exact against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from tests import gpu_util as G

pytestmark = pytest.mark.gpu

MFMA = 2


@pytest.fixture(scope="module")
def B():
    import paper_2405_14642_amd as B
    return B


@pytest.fixture(scope="module")
def ctx(B):
    c = B.Context(0)
    yield c
    c.close()


def operands(seed, batch, n):
    """Uniform operands; every fifth all ones, every seventh with bytes 0x80
    and 0x7F (the extreme balanced digits, with carries through them)."""
    rng = np.random.default_rng(seed)
    a, b = (rng.integers(0, 2**32, (batch, n), dtype=np.uint32) for _ in range(2))
    a[::5] = 0xFFFFFFFF
    b[::5] = 0xFFFFFFFF
    a[3::7] = 0x80808080
    b[3::7] = 0x7F7F7F7F
    return a, b


def padded(x, off):
    """x on the device, starting `off` words into its buffer."""
    flat = G.to_dev(np.concatenate([np.zeros(off, np.uint32), x.ravel()]))
    return flat[off:].reshape(x.shape)


def differing(got, exp):
    return np.nonzero((got != exp).any(axis=1))[0][:8].tolist()


# tiles hold 32, 64 and 128 words of an operand; chunks 4; a wave 4, 2 or 1 products
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 16, 17, 29, 32, 33, 36, 61, 64, 65, 68, 125, 128])
def test_small_full(B, ctx, orc, n, off):
    for batch in (1, 2, 5, 1031):
        a, b = operands(n, batch, n)
        out = G.empty_dev((batch * 2 * n + off,), np.uint32)[off:].reshape(batch, 2 * n)
        B.bigmul(ctx, padded(a, off), padded(b, off), out, algo=MFMA)
        G.sync()
        assert differing(G.from_dev(out, np.uint32), orc.mul(a, b)) == [], (n, off, batch)


def test_small_ragged(B, ctx, orc):
    """Every size up to 128 words in one batch, twice over and shuffled, so
    that a wave meets longer and shorter instances in turn."""
    n = np.random.default_rng(3).permutation(np.repeat(np.arange(1, 129), 2))
    off = np.concatenate([[0], np.cumsum(n)[:-1]])
    a, b = (x[0] for x in operands(9, 1, int(n.sum())))
    a, b = a.copy(), b.copy()
    rng = np.random.default_rng(4)
    for i in range(0, len(n), 2):
        sl = slice(off[i], off[i] + n[i])
        a[sl] = rng.integers(0, 2**32, n[i], dtype=np.uint32)
        b[sl] = rng.integers(0, 2**32, n[i], dtype=np.uint32)
    out = G.empty_dev((2 * a.size,), np.uint32)
    B.bigmul_v(ctx, G.to_dev(a), G.to_dev(b), out, G.desc_dev(off, off, 2 * off, n), len(n), 32, algo=MFMA)
    G.sync()
    got = G.from_dev(out, np.uint32)
    for o, k in zip(off, n):
        exp = orc.mul(a[None, o:o + k], b[None, o:o + k])[0]
        assert (got[2 * o:2 * (o + k)] == exp).all(), int(k)
