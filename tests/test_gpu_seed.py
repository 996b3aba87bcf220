"""Seeding on the device against the oracle's initialisation: stream counts
around the streams of one wave, every state length, padded rows."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


@pytest.mark.parametrize("n", [1, 15, 16, 17, 67])
@pytest.mark.parametrize("mexp", workloads.SUPPORTED_MEXP)
def test_seeded_states_match_oracle(torch, mexp, n):
    print("case seed mexp=%d n=%d" % (mexp, n), flush=True)
    N = mtgp.state_words(mexp)
    params = workloads.make_params(mexp, n, 0x5EED0 + n)
    seeds = (workloads.splitmix64(np.arange(n, dtype=np.uint64), 0x5EED) >> np.uint64(32)
             ).astype(np.uint32)
    seeds[0] = 0
    stride = N + 5
    g = mtgp.Generators(params, seeds, stride=stride)
    for again in range(2):
        if again:
            g.d_states.fill_(-1)
            g.reseed()
        rows = g.d_states.cpu().numpy().view(np.uint32).reshape(n, stride)
        for k in range(n):
            assert np.array_equal(rows[k, :N], oracle.seed(int(seeds[k]), N)), (k, again)
        if again:
            assert (rows[:, N:] == 0xFFFFFFFF).all()   # the padding is not written
    g.close()
