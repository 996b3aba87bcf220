"""Launches with and without room for groups: batches that alternate on one
workspace, and plain calls of more mexp-3217 streams than run at once, over
every step width, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu

MEXP, N = 3217, 101


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


def test_batches_with_and_without_groups_in_turn(torch):
    print("case groups in turn", flush=True)
    widths = [2, 8, 20, 33, 50, 63, 64, 100]
    n = len(widths)
    p = workloads.make_params(MEXP, n, 0x6B01)
    p[:, 1] = [N - w if w < 100 else 1 for w in widths]
    seeds = np.arange(n, dtype=np.uint32)
    g = mtgp.Generators(p, seeds)
    states = [oracle.seed(int(s), N) for s in seeds]
    out = [torch.empty(300000, dtype=torch.int32, device="cuda") for _ in range(n)]
    plans = [[(k, k & 1, c - 13 * k, out[k]) for k in range(n)] for c in (300000, 5000)]
    ws = torch.empty(max(mtgp.batch_workspace_query(g.d_params, i) for i in plans),
                     dtype=torch.uint8, device="cuda")
    for turn in range(6):
        items = plans[turn & 1]
        g.batch(items, ws)
        for k in range(n):
            c = items[k][2]
            e, states[k] = oracle.generate(p[k], states[k], c, as_float=bool(k & 1))
            got = out[k][:c].cpu().numpy().view(np.uint32)
            assert np.array_equal(got, np.asarray(e).view(np.uint32)), (turn, widths[k])
    assert np.array_equal(g.states_host(), np.array(states))
    assert mtgp.batch_errors(ws) == 0
    g.close()


@pytest.mark.parametrize("dtype", [0, 1])
def test_plain_calls_of_many_streams(torch, dtype):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 8 * cus + 99
    print("case plain many mexp=3217 n=%d dtype=%d" % (n, dtype), flush=True)
    p = workloads.make_params(MEXP, n, 0x6B02)
    p[:, 1] = 1 + np.arange(n) % (N - 2)           # every step width, W = 2 .. 100
    p[99:130, 5:21] = (workloads.splitmix64(np.arange(31 * 16, dtype=np.uint64), 0x77)
                       >> np.uint64(32)).astype(np.uint32).reshape(31, 16)   # not linear
    seeds = np.arange(n, dtype=np.uint32)
    g = mtgp.Generators(p, seeds)
    states = {k: oracle.seed(int(seeds[k]), N) for k in list(range(130)) + [n - 1]}
    for count in (1, 63, 777):
        got = g.generate(count, dtype).cpu().numpy().view(np.uint32).reshape(n, count)
        after = g.states_host()
        for k in states:
            e, states[k] = oracle.generate(p[k], states[k], count, as_float=bool(dtype))
            assert np.array_equal(got[k], np.asarray(e).view(np.uint32)), (count, k)
            assert np.array_equal(after[k], states[k]), (count, k)
    g.close()
