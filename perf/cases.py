"""The work a user of the library has it do, as cases that can be timed.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same
ranges, ``prepare`` makes what a program holds before the call (operand and
result buffers on the GPU, the stream queue), ``run`` is one pass through the
public entry points, ``work`` what the pass cannot do without and ``exact``
the results by Python's own integers.

Kinds: ``add`` (bigadd), ``add_v`` (bigadd_v), ``add_large`` (bigadd_large),
``mul`` (bigmul), ``mul_v`` (bigmul_v), ``stream`` (StreamQueue),
``mul_large`` (bigmul_large), ``add6`` / ``low`` / ``poly`` (fused).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2405_14642_amd as B

_PROGRAMS = {"add6": B.PROG_ADD6, "low": B.PROG_MUL_LOW, "poly": B.PROG_POLY}
_ctx = None


def _context():
    """The one context a program keeps."""
    global _ctx
    if _ctx is None:
        _ctx = B.Context(0)
    return _ctx


def listed():
    return [
        # one 4096-bit product: the smallest call, where latency is all
        {"name": "mul_one_4k", "kind": "mul", "limb_bits": 32, "n": 128, "batch": 1},
        # many 1024-bit products (the smallest size of the mixed stream and the addition sweep)
        {"name": "mul_1k", "kind": "mul", "limb_bits": 32, "n": 32, "batch": 1 << 18},
        # the quadratic sizes' smallest, 4096 bits, as a large batch
        {"name": "mul_4k", "kind": "mul", "limb_bits": 32, "n": 128, "batch": 1 << 16},
        # an odd size in 64-bit limbs and an odd batch: a size no kernel is cut for
        {"name": "mul_10k_odd", "kind": "mul", "limb_bits": 64, "n": 157, "batch": 3001},
        # 2^15 bits: the largest quadratic and the smallest transform size
        {"name": "mul_32k", "kind": "mul", "limb_bits": 32, "n": 1024, "batch": 4096},
        # 2^18 bits: the largest integer of a batch, few of them
        {"name": "mul_256k", "kind": "mul", "limb_bits": 32, "n": 8192, "batch": 64},
        # batched addition with carries out, 2^12 bits in 64-bit limbs
        {"name": "add_4k", "kind": "add", "limb_bits": 64, "n": 64, "batch": 1 << 18},
        # the same-length product (mod 2^N), 2^14 bits
        {"name": "low_16k", "kind": "low", "limb_bits": 64, "n": 256, "batch": 1 << 14},
        # the polynomial program at 2^16 bits: the largest case
        {"name": "poly_64k", "kind": "poly", "limb_bits": 64, "n": 1024, "batch": 4096},
        # bursts of mixed sizes (2^10 .. 2^18 bits) through the stream queue
        {"name": "stream_mixed", "kind": "stream", "limb_bits": 32, "lo": 10.0, "hi": 18.0, "count": 8000, "bursts": 8},
        # one product of 2^22-bit operands
        {"name": "mul_large_4m", "kind": "mul_large", "limb_bits": 32, "n": 1 << 17, "batch": 1},
        # one addition of 2^28-bit integers
        {"name": "add_large_256m", "kind": "add_large", "limb_bits": 32, "n": 1 << 23, "batch": 1},
    ]


def _log(rng, lo, hi):
    return max(int(lo), min(int(hi), round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(["mul", "mul", "mul", "mul", "add", "add", "add6", "low", "low", "poly", "poly", "mul_v", "stream",
                       "add_v", "mul_large", "add_large"])
    w = rng.choice([32, 64])
    q = w // 32
    c = {"kind": kind, "limb_bits": w}
    if kind in ("mul_v", "stream", "add_v"):
        c["lo"] = round(rng.uniform(8.0, 12.0), 2)
        c["hi"] = round(rng.uniform(13.0, 18.0), 2)
        c["count"] = _log(rng, 100, 8000)
        c["bursts"] = rng.randint(1, 8) if kind == "stream" else 1
        return c
    if kind in ("mul_large", "add_large"):
        top = 1 << 18 if kind == "mul_large" else 1 << 23
        c["n"] = _log(rng, 8200, top) // q
        c["batch"] = 1
        return c
    # sizes over the whole range, half of them any number, half a multiple of 8 words
    n32 = _log(rng, 2, 8192)
    if rng.random() < 0.5:
        n32 = max(8, n32 // 8 * 8)
    n32 = max(q, n32 // q * q)
    # words per operand, and products of words, that a pass may take
    most = (1 << 24) // n32
    if kind in ("mul", "low", "poly"):
        most = min(most, {"mul": 1 << 33, "low": 1 << 34, "poly": 1 << 33}[kind] // (n32 * n32))
    c["n"] = n32 // q
    c["batch"] = _log(rng, 1, max(1, min(most, 1 << 18)))
    return c


# ------------------------------------------------------------------ inputs
def _limbs(g, shape, limb_bits):
    if limb_bits == 32:
        return torch.randint(-(1 << 31), 1 << 31, shape, generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    hi = torch.randint(-(1 << 31), 1 << 31, shape, generator=g, device="cuda", dtype=torch.int64)
    lo = torch.randint(0, 1 << 32, shape, generator=g, device="cuda", dtype=torch.int64)
    return (hi << 32) | lo


def _sizes(c):
    """Limb counts of the case's ragged batch, log-uniform in [2^lo, 2^hi] bits."""
    r = np.random.RandomState(c["count"])
    return np.maximum(1, np.rint(np.exp2(r.uniform(c["lo"], c["hi"], c["count"])) / c["limb_bits"])).astype(np.int64)


def _operands(c, seed):
    """(a, b, sizes): uniform limbs, some operands carry-heavy.  Additions: a
    quarter of the instances has a all ones and b = 1, so that the carry runs
    the whole length; mixed batches: a tenth all ones; one large addition:
    uniform."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind, w = c["kind"], c["limb_bits"]
    if "n" in c:
        shape = (c["n"],) if kind in ("mul_large", "add_large") else (c["batch"], c["n"])
        a, b = _limbs(g, shape, w), _limbs(g, shape, w)
        if kind in ("add", "add6"):
            heavy = torch.rand(c["batch"], generator=g, device="cuda") < 0.25
            a[heavy] = -1
            b[heavy] = 0
            b[heavy, 0] = 1
        return a, b, None
    n = _sizes(c)
    total = int(n.sum())
    a, b = _limbs(g, (total,), w), _limbs(g, (total,), w)
    ones = torch.from_numpy(np.random.RandomState(seed % (1 << 32)).rand(len(n)) < 0.1).to("cuda")
    mask = torch.repeat_interleave(ones, torch.from_numpy(n).to("cuda"))
    a[mask] = -1
    b[mask] = -1
    return a, b, n


def prepare(c, seed):
    kind = c["kind"]
    a, b, sizes = _operands(c, seed)
    s = {"kind": kind, "ctx": _context(), "a": a, "b": b, "limb_bits": c["limb_bits"]}
    if sizes is not None:
        f = 1 if kind == "add_v" else 2
        d = np.zeros(len(sizes), dtype=B.DESC_DTYPE)
        off = np.concatenate([[0], np.cumsum(sizes)[:-1]])
        d["a_off"], d["b_off"], d["out_off"], d["n_limbs"] = off, off, f * off, sizes
        s["out"] = torch.empty(f * a.numel(), dtype=a.dtype, device="cuda")
        s["count"] = len(d)
        if kind == "stream":
            s["bursts"] = np.array_split(d, c["bursts"])
            s["queue"] = B.StreamQueue(s["ctx"], a, b, s["out"], c["limb_bits"], max(len(x) for x in s["bursts"]),
                                       use_graph=False)
        else:
            s["desc"] = torch.from_numpy(d.view(np.uint8).copy()).to("cuda")
            s["carry"] = torch.empty(len(d), dtype=torch.uint8, device="cuda") if kind == "add_v" else None
        return s
    if kind in ("add", "add_large"):
        s["out"] = torch.empty_like(a)
        s["carry"] = torch.empty(c["batch"], dtype=torch.uint8, device="cuda")
    elif kind in ("mul", "mul_large"):
        s["out"] = torch.empty(a.shape[:-1] + (2 * a.shape[-1],), dtype=a.dtype, device="cuda")
    else:
        s["out"] = torch.empty_like(a)
    return s


def run(s):
    kind, ctx, a, b, out = s["kind"], s["ctx"], s["a"], s["b"], s["out"]
    if kind == "mul":
        return B.bigmul(ctx, a, b, out)
    if kind == "add":
        return B.bigadd(ctx, a, b, out, s["carry"]), s["carry"]
    if kind in _PROGRAMS:
        return B.fused(ctx, _PROGRAMS[kind], a, b, out)
    if kind == "mul_v":
        return B.bigmul_v(ctx, a, b, out, s["desc"], s["count"], s["limb_bits"])
    if kind == "add_v":
        return B.bigadd_v(ctx, a, b, out, s["carry"], s["desc"], s["count"], s["limb_bits"]), s["carry"]
    if kind == "stream":  # the caller's stream waits for every burst
        for d in s["bursts"]:
            s["queue"].submit(d)
        return out
    if kind == "mul_large":
        return B.bigmul_large(ctx, a, b, out)
    return B.bigadd_large(ctx, a, b, out, s["carry"]), s["carry"]


# -------------------------------------------------------------- what it takes
def _product_ops(n32, low=False):
    """Operations of one product: the convolution of 8-bit digits, or six
    transforms modulo word-size primes where those are fewer."""
    d = 4 * n32
    school = d * d if low else 2 * d * d
    log = max(11, math.ceil(math.log2(4 * n32)))
    return min(school, 6 * (1 << (log - 1)) * log * 12)


def work(c):
    kind, q = c["kind"], c["limb_bits"] // 32
    sizes = _sizes(c) * q if "n" not in c else [c["n"] * q] * c["batch"]
    words = int(sum(int(x) for x in sizes)) if "n" not in c else c["n"] * q * c["batch"]
    reads, writes = 8 * words, 4 * words * (2 if kind in ("mul", "mul_v", "stream", "mul_large") else 1)
    if kind in ("add", "add_v", "add_large"):
        ops = words
        writes += c.get("batch", len(sizes))
    elif kind == "add6":
        ops = 6 * words
    elif "n" in c:
        ops = c["batch"] * _product_ops(c["n"] * q, kind in ("low", "poly")) * (4 if kind == "poly" else 1)
    else:
        ops = sum(_product_ops(int(x)) for x in sizes)
    return {"bytes": reads + writes, "flops": ops}


def _cost(c):
    """Rough seconds of exact() on one CPU core."""
    q = c["limb_bits"] // 32
    bits = [32.0 * q * c["n"]] if "n" in c else [float(x) * c["limb_bits"] for x in _sizes(c)]
    each = sum(1e-6 + b * 2e-10 + (0 if c["kind"].startswith("add") else 6e-9 * (b / 32) ** 1.585) for b in bits)
    return each * (4 if c["kind"] == "poly" else 1) * c.get("batch", 1) + 4e-9 * sum(bits) * c.get("batch", 1) / 32


def exact(c, seed):
    if _cost(c) > 15:
        return None
    kind, w = c["kind"], c["limb_bits"]
    a, b, sizes = _operands(c, seed)
    dt, shape = a.cpu().numpy().dtype, tuple(a.shape)
    a, b = a.cpu().numpy().tobytes(), b.cpu().numpy().tobytes()
    if sizes is None:
        sizes = [c["n"]] * c["batch"]
    out, carry, at = [], [], 0
    for n in sizes:
        nb = int(n) * w // 8
        x, y = int.from_bytes(a[at:at + nb], "little"), int.from_bytes(b[at:at + nb], "little")
        at += nb
        m = (1 << (8 * nb)) - 1
        if kind in ("add", "add_v", "add_large"):
            out.append(((x + y) & m).to_bytes(nb, "little"))
            carry.append((x + y) >> (8 * nb))
        elif kind == "add6":
            out.append(((4 * x + 3 * y) & m).to_bytes(nb, "little"))
        elif kind == "low":
            out.append((x * y & m).to_bytes(nb, "little"))
        elif kind == "poly":
            out.append(((((x * x + y) & m) * ((y * y + y) & m) + x * y) & m).to_bytes(nb, "little"))
        else:
            out.append((x * y).to_bytes(2 * nb, "little"))
    o = np.frombuffer(b"".join(out), dtype=dt)
    if kind in ("mul", "mul_large"):
        o = o.reshape(shape[:-1] + (2 * shape[-1],))
    elif "n" in c:
        o = o.reshape(shape)
    if kind in ("add", "add_v", "add_large"):
        return o, np.array(carry, dtype=np.uint8)
    return o
