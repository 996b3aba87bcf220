"""A stream's cached jump powers x^(c*lseg-1) mod p: their values against
Python integers, segment lengths that alternate without being built again,
sets that grow while a plan holds them, and the bound on what is kept."""
from __future__ import annotations

import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1501_07701_amd", "csrc")
U64 = ctypes.c_ulonglong


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("powers") / "powers_shim.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-mpclmul", "-shared", "-fPIC", "-I", CSRC,
                    os.path.join(ROOT, "tests", "shims", "powers_shim.cpp"),
                    os.path.join(CSRC, "mtgp_poly.cpp"), "-o", so], check=True)
    s = ctypes.CDLL(so)
    s.powers_new.restype = ctypes.c_void_p
    s.powers_delete.argtypes = [ctypes.c_void_p]
    s.powers_get.argtypes = [ctypes.c_void_p, U64, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    s.powers_hold.argtypes = [ctypes.c_void_p, U64, ctypes.c_int]
    s.powers_held.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    for f in (s.powers_built, s.powers_bytes):
        f.restype, f.argtypes = U64, [ctypes.c_void_p]
    s.powers_keep.restype = U64
    return s


def _mulmod(a, b, p, d):
    r = 0
    while b:
        if b & 1:
            r ^= a
        a <<= 1
        if a >> d & 1:
            a ^= p
        b >>= 1
    return r


def _powx(e, p, d):
    r, x = 1, 2 if d > 1 else 2 ^ p
    while e:
        if e & 1:
            r = _mulmod(r, x, p, d)
        x = _mulmod(x, x, p, d)
        e >>= 1
    return r


class Cache:
    def __init__(self, shim, d, seed):
        self.s, self.d = shim, d
        self.p = random.Random(seed).getrandbits(d) | 1 | 1 << d
        n = d // 64 + 1
        words = (U64 * n)(*[self.p >> (64 * i) & (2**64 - 1) for i in range(n)])
        self.c = shim.powers_new(words, n)
        self.words = (d + 31) // 32

    def get(self, lseg, n, power=0):
        """Power `power` of the set, and whether all n were there."""
        buf = (ctypes.c_uint32 * self.words)()
        there = self.s.powers_get(self.c, lseg, n, power, buf if power else None)
        return sum(v << (32 * i) for i, v in enumerate(buf)), there

    def want(self, lseg, c):
        return _powx(c * lseg - 1, self.p, self.d)


@pytest.mark.parametrize("d", [2, 31, 32, 63, 64, 65, 321])
def test_values(shim, d):
    c = Cache(shim, d, d)
    for lseg in (256, 1000, 65536):
        for power in (1, 2, 3, 7):
            assert c.get(lseg, 7, power)[0] == c.want(lseg, power), (lseg, power)
    # fewer are there, more are appended
    assert c.get(1000, 3, 3) == (c.want(1000, 3), 1)
    assert c.get(1000, 9, 9) == (c.want(1000, 9), 0)
    shim.powers_delete(c.c)


def test_alternating_lengths_are_built_once(shim):
    """Small and large batches in turn, and requests of many lengths."""
    c = Cache(shim, 3217, 7)
    lengths = [16384, 24576, 32768, 49152, 65536, 98304, 131072, 69632]
    for lseg in lengths:
        assert c.get(lseg, 16)[1] == 0
    before = shim.powers_built(c.c)
    assert before == 16 * len(lengths)
    rng = random.Random(3)
    for _ in range(200):
        assert c.get(rng.choice(lengths), rng.randint(1, 16))[1] == 1
    assert shim.powers_built(c.c) == before
    shim.powers_delete(c.c)


def test_held_sets_do_not_change(shim):
    c = Cache(shim, 321, 9)
    buf = (ctypes.c_uint32 * c.words)()
    shim.powers_hold(c.c, 512, 4)
    c.get(512, 40)
    for lseg in range(1024, 1024 + 600):       # the first set is long gone
        c.get(lseg, 4)
    assert c.get(512, 1)[1] == 0
    assert shim.powers_held(c.c, 0, 4, buf) == 4
    assert sum(v << (32 * i) for i, v in enumerate(buf)) == c.want(512, 4)
    shim.powers_delete(c.c)


def test_what_is_kept_is_bounded(shim):
    c = Cache(shim, 3217, 5)
    one = 4 * c.words
    keep = shim.powers_keep()
    for lseg in range(300, 300 + 40):
        c.get(lseg, 16)
        assert shim.powers_bytes(c.c) <= 16 * one + keep
    # a set larger than that leaves room for one more of its size
    n = int(2 * keep / one)
    c.get(4096, n)
    c.get(5120, n)
    assert shim.powers_bytes(c.c) <= 2 * n * one
    assert c.get(4096, n)[1] == 1 and c.get(5120, n)[1] == 1
    shim.powers_delete(c.c)
