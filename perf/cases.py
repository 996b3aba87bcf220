"""Performance cases of the MTGP32 generator: what a program has it do.

Every case goes through the public entry points of
``paper_1501_07701_amd.mtgp``: plain bulk generation, batched generation
(long streams split by jump-ahead), the device-side draw API, the screening
counts and the serving loop, over the four exponents, both output types,
and sizes from a few hundred numbers to billions.  Parameter sets are drawn
as in the repository's workloads: pos uniform in [1, N-2], shifts uniform
in [0, 31], tables spanned by random basis words.  Generators continue from
pass to pass, as in a program that draws again and again; cases with
``reseed`` go back to the seed status first, as a program does that starts
its next replication.
"""
import math

import numpy as np
import torch

from paper_1501_07701_amd import mtgp

MEXPS = (3217, 11213, 23209, 44497)


def listed():
    return [
        # the smallest call: a simulation of a few thread groups asks for its
        # next numbers; launch and latency are all there is
        {"name": "plain_small_u32", "kind": "plain", "mexp": 11213, "streams": 8, "count": 256,
         "dtype": "u32", "reseed": False},
        # one replication of 1,000 statuses of period 2^3217: seed, then an
        # odd number of floats each
        {"name": "plain_f32_3217", "kind": "plain", "mexp": 3217, "streams": 1000, "count": 5003,
         "dtype": "f32", "reseed": True},
        # every resident stream of a large simulation advances a little:
        # states are a large part of the traffic
        {"name": "plain_u32_11213", "kind": "plain", "mexp": 11213, "streams": 16384,
         "count": 1000, "dtype": "u32", "reseed": False},
        # long states, ragged counts, floats: an ordinary Monte Carlo call
        {"name": "plain_f32_44497", "kind": "plain", "mexp": 44497, "streams": 1024,
         "count": 12289, "dtype": "f32", "reseed": True},
        # the 128 statuses of Saito's sample, 2^24 numbers each (the
        # repository's headline batch)
        {"name": "batch_u32_11213", "kind": "batch", "mexp": 11213, "streams": 128,
         "log2_lo": 24.0, "log2_hi": 24.0, "dtype": "u32", "reseed": True},
        # a middling batch: few streams, a million floats each
        {"name": "batch_f32_11213_mid", "kind": "batch", "mexp": 11213, "streams": 100,
         "log2_lo": 19.93, "log2_hi": 19.93, "dtype": "f32", "reseed": False},
        # 4,096 statuses of period 2^23209, 2^20 numbers each in one batch
        {"name": "batch_u32_23209", "kind": "batch", "mexp": 23209, "streams": 4096,
         "log2_lo": 20.0, "log2_hi": 20.0, "dtype": "u32", "reseed": False},
        # uneven requests of both types, lengths log-uniform in [2^10, 2^22]
        {"name": "batch_mixed_44497", "kind": "batch", "mexp": 44497, "streams": 512,
         "log2_lo": 10.0, "log2_hi": 22.0, "dtype": "mixed", "reseed": False},
        # the paper's 10,000 statuses of period 2^3217, all short steps
        {"name": "batch_u32_3217", "kind": "batch", "mexp": 3217, "streams": 10000,
         "log2_lo": 18.0, "log2_hi": 18.0, "dtype": "u32", "reseed": True},
        # gap and Hamming-weight counts of generated numbers
        {"name": "screen_3217", "kind": "screen", "mexp": 3217, "streams": 4000,
         "count": 131072, "log2_gap": 30, "bins": 16},
        # a kernel's thread groups draw from their own streams
        {"name": "draws_u32_11213", "kind": "draws", "mexp": 11213, "streams": 512,
         "count": 32768, "dtype": "u32", "threads": 256, "reseed": False},
        # a burst of requests against resident streams through the server
        {"name": "serve_mixed_11213", "kind": "serve", "mexp": 11213, "streams": 256,
         "requests": 1000, "log2_lo": 8.0, "log2_hi": 20.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "plain", "plain", "batch", "batch", "screen", "draws", "serve"])
    mexp = rng.choice(MEXPS)
    c = {"kind": kind, "mexp": mexp}
    if kind == "plain":
        c["streams"] = _log_int(rng, 4, 16384)
        # at most 2^27 numbers; a stream's steps follow one another, so a
        # plain call does not ask one stream for very many
        c["count"] = _log_int(rng, 200, min(20000, (1 << 27) // c["streams"]))
        c["dtype"] = rng.choice(["u32", "f32"])
        c["reseed"] = rng.random() < 0.5
    elif kind == "batch":
        c["streams"] = _log_int(rng, 48, 4096)
        # lengths up to 2^22, at most 2^30 numbers in all; half of the
        # batches are even, half log-uniform over some octaves
        hi = min(22.0, 30.0 - math.log2(c["streams"]))
        hi = rng.uniform(min(17.0, hi - 1.0), hi)
        c["log2_hi"] = round(hi, 3)
        c["log2_lo"] = c["log2_hi"] if rng.random() < 0.5 else round(rng.uniform(8.0, hi), 3)
        c["dtype"] = rng.choice(["u32", "f32", "mixed"])
        c["reseed"] = rng.random() < 0.5
    elif kind == "screen":
        c["streams"] = _log_int(rng, 100, 10000)
        c["count"] = _log_int(rng, 1000, min(1 << 20, (1 << 29) // c["streams"]))
        c["log2_gap"] = rng.randint(27, 31)
        c["bins"] = rng.choice([8, 16, 33, 64])
    elif kind == "draws":
        c["streams"] = _log_int(rng, 16, 2048)
        c["count"] = _log_int(rng, 500, 40000)
        c["dtype"] = rng.choice(["u32", "f32"])
        c["threads"] = rng.choice([64, 128, 256, 512])
        c["reseed"] = rng.random() < 0.5
    else:
        c["mexp"] = rng.choice([3217, 11213])
        c["streams"] = _log_int(rng, 64, 256)
        c["requests"] = _log_int(rng, 100, 1000)
        c["log2_lo"] = 8.0
        c["log2_hi"] = round(rng.uniform(14.0, 20.0), 3)
    return c


# ---------------------------------------------------------------- inputs --

def _span(basis):
    """(n, 4) basis words -> (n, 16) table: entry i is the XOR of the words
    that the bits of i select."""
    tbl = np.zeros((basis.shape[0], 16), dtype=np.uint32)
    for i in range(16):
        for b in range(4):
            if (i >> b) & 1:
                tbl[:, i] ^= basis[:, b]
    return tbl


def _inputs(case, seed):
    """(params (n, 53), seeds (n,)) of a case."""
    n, mexp = case["streams"], case["mexp"]
    words = mexp // 32 + 1
    rng = np.random.default_rng([seed, 7701])
    p = np.zeros((n, 53), dtype=np.uint32)
    p[:, 0] = mexp
    p[:, 1] = rng.integers(1, words - 1, n)          # [1, N-2]
    p[:, 2] = rng.integers(0, 32, n)
    p[:, 3] = rng.integers(0, 32, n)
    p[:, 4] = (0xFFFFFFFF << (32 * words - mexp)) & 0xFFFFFFFF
    p[:, 5:21] = _span(rng.integers(0, 1 << 32, (n, 4), dtype=np.uint32))
    tmp = _span(rng.integers(0, 1 << 32, (n, 4), dtype=np.uint32))
    p[:, 21:37] = tmp
    p[:, 37:53] = np.uint32(0x3F800000) | (tmp >> np.uint32(9))
    return p, rng.integers(0, 1 << 32, n, dtype=np.uint32)


def _lengths(case, seed, n):
    """Lengths and types (0: uint32, 1: float32) of n requests: the case's
    own requests, in an order that the seed gives."""
    lo, hi = case["log2_lo"], case["log2_hi"]
    u = (np.arange(n) + 0.5) / n
    length = np.floor(np.exp2(lo + (hi - lo) * u))
    kind = {"u32": np.zeros(n), "f32": np.ones(n)}.get(case.get("dtype", "mixed"))
    dtype = np.arange(n) % 2 if kind is None else kind
    order = np.random.default_rng([seed, 7702]).permutation(n)
    return length[order].astype(np.int64), dtype[order].astype(np.int32)


def _places(length, dtype):
    """Offset of each request in the buffer of its type, and the buffers'
    sizes; requests follow one another on whole cache lines."""
    off = np.zeros(len(length), dtype=np.int64)
    size = [0, 0]
    for i, (m, d) in enumerate(zip(length, dtype)):
        off[i] = size[d]
        size[d] += (int(m) + 31) // 32 * 32
    return off, size


class State:
    """What a program holds: its generators, buffers and, for a server, the
    server, which it closes."""

    srv = None

    def __del__(self):
        if self.srv is not None:
            self.srv.close()
        if getattr(self, "g", None) is not None:
            self.g.close()


def prepare(case, seed):
    s = State()
    kind = case["kind"]
    params, seeds = _inputs(case, seed)
    s.kind, s.reseed = kind, case.get("reseed", False)
    s.g = g = mtgp.Generators(params, seeds)
    if kind in ("plain", "draws"):
        s.count = case["count"]
        s.dtype = mtgp.F32 if case["dtype"] == "f32" else mtgp.U32
        s.threads = case.get("threads")
        s.out = torch.empty(g.n * s.count, device="cuda",
                            dtype=torch.float32 if s.dtype == mtgp.F32 else torch.int32)
    elif kind == "screen":
        s.n, s.count, s.bins = g.n, case["count"], case["bins"]
        s.lo, s.hi = 0, 1 << case["log2_gap"]
        s.words = g.generate(s.count, mtgp.U32)
        s.counts = torch.empty(g.n * (s.bins + 9), dtype=torch.int64, device="cuda")
    else:
        n = g.n if kind == "batch" else case["requests"]
        length, dtype = _lengths(case, seed, n)
        off, size = _places(length, dtype)
        # gaps between requests stay zero
        buf = [torch.zeros(size[0], dtype=torch.int32, device="cuda"),
               torch.zeros(size[1], dtype=torch.float32, device="cuda")]
        at = [buf[d].data_ptr() + 4 * int(o) for d, o in zip(dtype, off)]
        s.out = [b for b in buf if b.numel()]
        if kind == "batch":
            items = [(k, int(dtype[k]), int(length[k]), at[k]) for k in range(n)]
            s.ws = g.workspace(items)
            s.items = mtgp.make_work(items)
        else:
            rng = np.random.default_rng([seed, 7703])
            s.arrive = np.zeros(n, dtype=np.uint64)
            s.stream = rng.integers(0, g.n, n).astype(np.int32)
            s.length, s.dtype, s.keep = length.astype(np.uint64), dtype, at
            # a service is warmed up: every resident stream's jump-ahead
            # polynomial is there before the first request
            mtgp.stream_polynomials(g.d_params, g.n, g.mexp)
            s.srv = mtgp.Server(g, 2 << 30, inflight=8, max_batch_items=128,
                                batch_window_ns=20000, workspace_bytes_per_batch=32 << 20)
    return s


def run(s):
    g = s.g
    if s.reseed:
        g.reseed()
    if s.kind == "plain":
        g.generate(s.count, s.dtype, out=s.out)
    elif s.kind == "draws":
        mtgp.generate_workgroup(g.d_params, g.d_states, g.stride, g.n, s.count, s.out, s.dtype,
                                s.threads)
    elif s.kind == "batch":
        mtgp.generate_batch(g.d_params, g.d_states, g.stride, s.items, s.ws)
    elif s.kind == "serve":
        s.srv.replay(s.arrive, s.stream, s.length, s.dtype, keep=s.keep)
    else:
        mtgp.screen(s.words, s.n, s.count, s.lo, s.hi, s.bins, s.counts)
        return s.counts
    return [s.out, g.d_states]


def work(case):
    n, words = case["streams"], case["mexp"] // 32 + 1
    if case["kind"] == "screen":
        return {"bytes": n * case["count"] * 4 + n * (case["bins"] + 9) * 8, "flops": 0}
    if case["kind"] in ("plain", "draws"):
        outputs = n * case["count"]
    else:
        lo, hi = case["log2_lo"], case["log2_hi"]
        mean = 2.0 ** hi if hi == lo else (2.0 ** hi - 2.0 ** lo) / ((hi - lo) * math.log(2.0))
        outputs = case.get("requests", n) * mean
    # the numbers, each stream's parameters, and its state read (unless it
    # is seeded anew) and written
    state = n * (4 * words * (1 if case.get("reseed") else 2) + 256)
    return {"bytes": int(outputs * 4 + state), "flops": 0}


# ------------------------------------------------------------- in 64 bits --

def exact(case, seed):
    """The definition itself, word after word, all streams at once."""
    if case["kind"] not in ("plain", "draws") or case["count"] > 40000:
        return None
    if case["count"] * case["streams"] > 1 << 25:
        return None
    params, seeds = _inputs(case, seed)
    n, count, words = case["streams"], case["count"], case["mexp"] // 32 + 1
    p = params.astype(np.int64)
    M = 0xFFFFFFFF
    x = np.zeros((words + count, n), dtype=np.int64)
    x[0] = seeds
    for i in range(1, words):
        x[i] = (1812433253 * (x[i - 1] ^ (x[i - 1] >> 30)) + i) & M
    pos, sh1, sh2, mask = p[:, 1], p[:, 2], p[:, 3], p[:, 4]
    k = np.arange(n)
    f32 = case["dtype"] == "f32"
    out = np.zeros((n, count), dtype=np.float64 if f32 else np.int64)
    for j in range(count):
        X = (x[j] & mask) ^ x[j + 1]
        X ^= (X << sh1) & M
        Y = X ^ (x[j + pos, k] >> sh2)
        new = Y ^ p[k, 5 + (Y & 15)]
        x[j + words] = new
        H = x[j + pos - 1, k]
        H = H ^ (H >> 16)
        H = H ^ (H >> 8)
        t = H & 15
        if f32:
            out[:, j] = (((new >> 9) ^ p[k, 37 + t]) & 0x7FFFFF) / float(1 << 23)
        else:
            out[:, j] = new ^ p[k, 21 + t]
    states = x[count:].T.astype(np.uint32).view(np.int32).astype(np.int64)
    if not f32:
        out = out.astype(np.uint32).view(np.int32).astype(np.int64)
    return [out.reshape(-1), states.reshape(-1)]
