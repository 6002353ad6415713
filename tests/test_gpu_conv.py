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


# one straight-line wave takes up to 256, 384, 512 and 640 words, two 768 and
# (above 896) 1024; workgroups of 4, 8 and 16 waves 896, 2048 and 4096, one of
# 16 waves with two units each 8192; a tile is 32 words of an operand, a unit
# of the loops 256; a chunk is 4 words
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("n", [129, 160, 161, 253, 255, 256, 257, 288, 289, 381, 384, 385, 480, 481, 509, 512, 513, 545,
                               637, 640, 641, 767, 768, 769, 893, 896, 897, 992, 1021, 1024, 1025, 1057, 1536, 1537,
                               2016, 2047, 2048, 2049, 3073, 4064, 4093, 4096, 4097, 6145, 8160, 8191, 8192])
def test_workgroup_full(B, ctx, orc, n, off):
    batch = 13 if n <= 1100 else 4
    a, b = operands(n, batch, n)
    out = G.empty_dev((batch * 2 * n + off,), np.uint32)[off:].reshape(batch, 2 * n)
    B.bigmul(ctx, padded(a, off), padded(b, off), out, algo=MFMA)
    G.sync()
    assert differing(G.from_dev(out, np.uint32), orc.mul(a, b)) == []


def test_workgroup_many(B, ctx, orc):
    """More products than resident workgroups, so that each meets several."""
    for n, batch in ((200, 33001), (300, 25003), (500, 25001), (600, 17001), (700, 13001), (800, 9001), (1000, 9001)):
        a, b = operands(n, batch, n)
        out = G.empty_dev((batch, 2 * n), np.uint32)
        B.bigmul(ctx, G.to_dev(a), G.to_dev(b), out, algo=MFMA)
        G.sync()
        pick = np.unique(np.r_[:40, np.linspace(0, batch - 1, 500).astype(int), batch - 40:batch])
        assert differing(G.from_dev(out, np.uint32)[pick], orc.mul(a[pick], b[pick])) == [], n


@pytest.mark.parametrize("sizes", [np.arange(1, 129), np.r_[129:257:3, 257:513:7, 513:1025:19],
                                   np.r_[1025:2049:101, 2049:4097:307, 4097:8193:1023]], ids=["small", "mid", "large"])
def test_ragged(B, ctx, orc, sizes):
    """Sizes of every class twice over and shuffled, each instance on a wave or
    workgroup of its own."""
    n = np.random.default_rng(3).permutation(np.repeat(sizes, 2))
    off = np.concatenate([[0], np.cumsum(n)[:-1]])
    rng = np.random.default_rng(4)
    a, b = (rng.integers(0, 2**32, int(n.sum()), dtype=np.uint32) for _ in range(2))
    for i in range(0, len(n), 3):
        a[off[i]:off[i] + n[i]] = 0xFFFFFFFF
        b[off[i]:off[i] + n[i]] = 0xFFFFFFFF
    out = G.empty_dev((2 * a.size,), np.uint32)
    B.bigmul_v(ctx, G.to_dev(a), G.to_dev(b), out, G.desc_dev(off, off, 2 * off, n), len(n), 32, algo=MFMA)
    G.sync()
    got = G.from_dev(out, np.uint32)
    for o, k in zip(off, n):
        exp = orc.mul(a[None, o:o + k], b[None, o:o + k])[0]
        assert (got[2 * o:2 * (o + k)] == exp).all(), int(k)


PROG_POLY, PROG_MUL_LOW = 2, 3


# tiles hold 64, 128 and 256 words of a low product's operand; one wave takes
# 512, 768 and 1024 words, workgroups of 3 (Poly), 4, 8 and 16 waves 1536 ..
# 8192; instances of up to 32 words run elsewhere
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("n", [32, 33, 61, 64, 65, 127, 128, 129, 197, 253, 256, 257, 300, 509, 512, 513, 577, 767, 768,
                               769, 1021, 1024, 1025, 1531, 1536, 1537, 1600, 2045, 2048, 2049, 3333, 4096, 4097, 6000, 8189, 8192])
def test_low_and_poly(B, ctx, n, off):
    import oracle as O
    batch = 23 if n <= 512 else 5 if n <= 2048 else 2
    a, b = operands(n, batch, n)
    for prog, want in ((PROG_MUL_LOW, O.mul_low), (PROG_POLY, O.poly)):
        out = G.empty_dev((batch * n + off,), np.uint32)[off:].reshape(batch, n)
        B.fused(ctx, prog, padded(a, off), padded(b, off), out)
        G.sync()
        assert differing(G.from_dev(out, np.uint32), want(a, b)) == [], prog


VALU = 1


# an instance takes 1, 2, 4 .. 32 lanes of two result words each
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32])
def test_packed_full(B, ctx, orc, n, off):
    for batch in (1, 3, 64, 20011):
        a, b = operands(n, batch, n)
        out = G.empty_dev((batch * 2 * n + off,), np.uint32)[off:].reshape(batch, 2 * n)
        B.bigmul(ctx, padded(a, off), padded(b, off), out, algo=VALU)
        G.sync()
        assert differing(G.from_dev(out, np.uint32), orc.mul(a, b)) == [], (n, off, batch)


# one workgroup bins up to 4096 descriptors, a grid of them more; a class may
# be absent, and the classes up to 128 words share one launch
@pytest.mark.parametrize("algo", [0, MFMA])
@pytest.mark.parametrize("sizes", [[5], [30, 100], [3, 20, 50, 120, 300]], ids=["one", "two", "five"])
@pytest.mark.parametrize("count", [1, 3, 1025, 4096, 4097])
def test_ragged_counts(B, ctx, orc, count, sizes, algo):
    n = np.random.default_rng(count).choice(sizes, count)
    off = np.concatenate([[0], np.cumsum(n)[:-1]])
    rng = np.random.default_rng(5)
    a, b = (rng.integers(0, 2**32, int(n.sum()), dtype=np.uint32) for _ in range(2))
    out = G.empty_dev((2 * a.size,), np.uint32)
    B.bigmul_v(ctx, G.to_dev(a), G.to_dev(b), out, G.desc_dev(off, off, 2 * off, n), len(n), 32, algo=algo)
    G.sync()
    got = G.from_dev(out, np.uint32)
    for k in sizes:
        at = off[n == k][:, None]
        rows, cols = at + np.arange(k), 2 * at + np.arange(2 * k)
        assert (got[cols] == orc.mul(a[rows], b[rows])).all() if at.size else True, k


def run_looping(B, ctx, orc, sizes, count, algo):
    """`count` products of shuffled sizes in one list: half of them of the
    first (largest) size, half of those all ones.  Descriptors share 24 operand
    pairs per size; every word of every result is compared, on the device."""
    import torch
    rng = np.random.default_rng(count)
    pairs, nmax = 24, max(sizes)
    a, b = (rng.integers(0, 2**32, (len(sizes) * pairs, nmax), dtype=np.uint32) for _ in range(2))
    a[:pairs // 2] = 0xFFFFFFFF
    b[:pairs // 2] = 0xFFFFFFFF
    exp = np.zeros((len(a), 2 * nmax), np.uint32)
    for i, n in enumerate(sizes):
        s = slice(i * pairs, (i + 1) * pairs)
        exp[s, :2 * n] = orc.mul(np.ascontiguousarray(a[s, :n]), np.ascontiguousarray(b[s, :n]))
    which = np.where(rng.random(count) < 0.5, 0, rng.integers(0, len(sizes), count))
    pair = which * pairs + rng.integers(0, pairs, count)
    out = torch.zeros((count, 2 * nmax), dtype=torch.int32, device="cuda")
    d = G.desc_dev(pair * nmax, pair * nmax, np.arange(count) * 2 * nmax, np.asarray(sizes)[which])
    B.bigmul_v(ctx, G.to_dev(a), G.to_dev(b), out, d, count, 32, algo=algo)
    G.sync()
    e, p = G.to_dev(exp), torch.from_numpy(pair).cuda()
    bad = torch.cat([(out[i:i + 4096] != e[p[i:i + 4096]]).any(dim=1) for i in range(0, count, 4096)])
    at = bad.nonzero().flatten().cpu().numpy()
    assert at.size == 0, f"{at.size} of {count} differ, of {np.unique(np.asarray(sizes)[which[at]]).tolist()} words"


# at least twice as many products as the waves or straight-line workgroups of
# any grid (4 * 256 per class up to 128 words, 8 times the resident ones above),
# so that each meets longer and shorter ones in turn
@pytest.mark.parametrize("sizes,count", [((16, 1, 13), 40000), ((32, 29, 17), 40000), ((64, 61, 33), 20000),
                                         ((128, 125, 65), 10000), ((256, 253, 200, 129), 70000),
                                         ((512, 509, 300, 257), 35000), ((1024, 1021, 600, 513), 18000)],
                         ids=lambda v: str(v[0]) if isinstance(v, tuple) else "")
def test_ragged_looping(B, ctx, orc, sizes, count):
    run_looping(B, ctx, orc, sizes, count, MFMA)


KARATSUBA = 5


# 81, 27 and 9 base products per instance, of sizes that follow the instance's
@pytest.mark.parametrize("sizes,base,count", [((8192, 8189, 6000, 4097), 512, 420), ((8192, 8189, 6000, 4097), 1024, 640),
                                              ((4096, 4093, 3000, 2049), 1024, 1900)])
def test_ragged_karatsuba_looping(B, orc, sizes, base, count):
    c = B.Context(0)
    try:
        B.tune_set_kara(c, [base] * B.NUM_CLASSES)
        run_looping(B, c, orc, sizes, count, KARATSUBA)
    finally:
        c.close()


# the sizes of workgroups of 8 and 16 waves (one or two units each), 12 and 16
# chunks apart among them: the digit areas of successive products then differ
# in length by as much as the waves' exchanged words lie apart
@pytest.mark.parametrize("sizes,count", [((2048, 2045, 2000, 1984, 1100, 1036), 9000), ((4096, 4093, 4048, 4032, 2100), 4500),
                                         ((8192, 8189, 8144, 8128, 4200), 4200)],
                         ids=lambda v: str(v[0]) if isinstance(v, tuple) else "")
def test_ragged_looping_waves(B, ctx, orc, sizes, count):
    run_looping(B, ctx, orc, sizes, count, MFMA)


def test_ragged_karatsuba_looping_waves(B, ctx, orc):
    """Nine base products of 1025 .. 2048 words per instance (the default base)."""
    run_looping(B, ctx, orc, (8192, 8189, 7936, 6000, 4097), 1100, KARATSUBA)


# Poly of 33 to 36 words: several to a wavefront on the VALU up to 1000 instances
@pytest.mark.parametrize("batch", [1, 999, 1000, 1001])
@pytest.mark.parametrize("n", [33, 35, 36, 37])
def test_poly_few(B, ctx, n, batch):
    import oracle as O
    a, b = operands(n + batch, batch, n)
    out = G.empty_dev((batch, n), np.uint32)
    B.fused(ctx, PROG_POLY, G.to_dev(a), G.to_dev(b), out)
    G.sync()
    assert differing(G.from_dev(out, np.uint32), O.poly(a, b)) == []
