"""Segment lengths of split requests: every member of a group gets its least
number of outputs, groups hold no more than they may, and requests of any
length name few segment lengths (each costs a stream's powers of x)."""
from __future__ import annotations

import ctypes
import math
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
U64 = ctypes.c_ulonglong


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("split") / "split_shim.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_1501_07701_amd", "csrc"),
                    os.path.join(ROOT, "tests", "shims", "split_shim.cpp"), "-o", so], check=True)
    s = ctypes.CDLL(so)
    s.split_segment_length.restype, s.split_segment_length.argtypes = U64, [U64]
    s.split_group_length.restype = s.split_group_least.restype = U64
    s.split_group_length.argtypes = [ctypes.c_uint, U64, U64, ctypes.c_int]
    s.split_group_least.argtypes = [ctypes.c_uint, ctypes.c_int]
    s.split_group_long_enough.argtypes = [ctypes.c_uint, U64, ctypes.c_int]
    return s


@pytest.mark.parametrize("floor", [128, 1024, 5000])
@pytest.mark.parametrize("w", [2, 8, 9, 16, 17, 32, 33, 63])
@pytest.mark.parametrize("steps", [1024, 1536, 6700, 1 << 20])
def test_group_lengths(shim, w, steps, floor):
    n = shim.split_group_members(w)
    item = max(steps, floor) * (60 + w)
    least = shim.split_group_least(w, floor)
    assert least >= 8192 and least >= 8 * floor and 2 * least >= (w - 1) * floor
    rng = random.Random(1000 * w + steps)
    counts = [int(2 ** rng.uniform(15, 24)) for _ in range(4000)]
    counts += [n * least, n * least + 1, n * least - 1, n // 2 * least, 2 * least, item, item + 1,
               2 * item, 2 * item + 1]
    lengths = {}
    for count in counts:
        if not shim.split_group_long_enough(w, count, floor):
            assert count < n * least
            continue
        lseg = shim.split_group_length(w, count, item, floor)
        segs = -(-count // lseg)
        items = -(-count // item)
        share = item // n if items > 2 else -(-count // (items * n))
        share = max(least, share)
        # at most a quarter over the share
        assert share <= lseg and 4 * lseg <= 5 * share
        # half the members of a first group are busy, but for the rounding
        assert 2 * segs >= n or lseg > least
        assert 5 * segs >= 2 * n
        lengths.setdefault(int(math.log2(count)), set()).add(lseg)
    for octave, found in lengths.items():
        assert len(found) <= 5, (octave, found)
    assert len(set().union(*lengths.values())) <= 4 * len(lengths) + 1
    # requests of more than two groups all share one length
    assert len({shim.split_group_length(w, c, item, floor) for c in counts if c > 2 * item}) == 1


def test_one_group_is_cut_evenly(shim):
    for w, want in ((2, 1 << 15), (8, 1 << 15), (16, 1 << 16), (32, 1 << 17), (40, 1 << 16)):
        assert shim.split_group_length(w, 1 << 18, 1 << 19, 1024) == want


def test_segment_length_grid(shim):
    for v in [1, 255, 256, 1023, 1024, 5000, 123456, 1 << 20, (1 << 31) + 12345]:
        got = shim.split_segment_length(v)
        assert got % 256 == 0 and got >= 256
        assert got <= max(v, 256) and 5 * got >= 4 * (v - 255)
