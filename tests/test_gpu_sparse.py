"""Batches of few items (wide streams by whole workgroups, the others by
waves) against the oracle: widths around the line between the two, both
types, lengths from one output to split requests, and numbers of items on
both sides of the rule."""
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


def _check(torch, g, p, seeds, counts, dts, look):
    n, N = p.shape[0], g.N
    off = np.concatenate([[0], np.cumsum(counts)])
    out = torch.empty(int(off[-1]), dtype=torch.int32, device="cuda")
    items = [(k, int(dts[k]), int(counts[k]), out.data_ptr() + 4 * int(off[k])) for k in range(n)]
    ws = g.workspace(items)
    states = {k: oracle.seed(int(seeds[k]), N) for k in look}
    for _ in range(2):
        g.batch(items, ws)
        got = out.cpu().numpy().view(np.uint32)
        after = g.states_host()
        for k in look:
            e, states[k] = oracle.generate(p[k], states[k], int(counts[k]), as_float=bool(dts[k]))
            assert np.array_equal(got[off[k]:off[k + 1]], np.asarray(e).view(np.uint32)), k
            assert np.array_equal(after[k], states[k]), k
    assert mtgp.batch_errors(ws) == 0


@pytest.mark.parametrize("mexp", [11213, 23209, 44497])
def test_widths_on_both_sides(torch, mexp):
    print("case sparse widths mexp=%d" % mexp, flush=True)
    N = mexp // 32 + 1
    widths = [2, 17, 47, 63, 64, 127, 128, 129, 191, 255, 256, 257, 319, N - 1, 130, 40]
    n = len(widths)
    p = workloads.make_params(mexp, n, 0x5A25)
    p[:, 1] = [N - w for w in widths]
    p[14:, 5:21] = (workloads.splitmix64(np.arange(32, dtype=np.uint64), 0xABD)
                    >> np.uint64(32)).astype(np.uint32).reshape(2, 16)   # not linear
    seeds = np.arange(n, dtype=np.uint32)
    counts = np.array([400000 - 37 * k if k % 3 else 1 + 997 * k for k in range(n)])
    counts[14:] = 3000
    g = mtgp.Generators(p, seeds)
    _check(torch, g, p, seeds, counts, np.arange(n) % 2, range(n))
    g.close()


@pytest.mark.parametrize("extra", [0, 1])
def test_numbers_of_items_around_the_rule(torch, extra):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 6 * cus + extra
    print("case sparse items n=%d" % n, flush=True)
    p = workloads.make_params(11213, n, 0x5A26)
    seeds = np.arange(n, dtype=np.uint32)
    g = mtgp.Generators(p, seeds)
    _check(torch, g, p, seeds, np.full(n, 1500), np.arange(n) % 2,
           [0, 1, n // 3, n // 2, n - 2, n - 1])
    g.close()
