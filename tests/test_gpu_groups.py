"""Groups: segments of one narrow stream run together on a wave.  Outputs,
final states and continuations against the oracle at every group size and
number of lanes per class, request lengths around the group thresholds (the
last segment short, full, or one output long), a workspace without room for
groups, and repairs among many requests."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu

N = 101
WIDTHS = [2, 3, 4, 5, 7, 8, 9, 12, 16, 17, 25, 32, 33, 64]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


def _streams(master):
    p = workloads.make_params(3217, len(WIDTHS), master)
    p[:, 1] = [N - w for w in WIDTHS]
    p[0, 3], p[1, 3], p[3, 3] = 0, 31, 1
    return p, np.arange(1, len(WIDTHS) + 1, dtype=np.uint32)


@pytest.mark.parametrize("count", [2 * 16384, 4 * 16384 - 1, 4 * 16384 + 1, 8 * 16384, 150001,
                                   300000])
def test_groups_match_oracle(torch, count):
    print("case groups count=%d" % count, flush=True)
    p, seeds = _streams(0x6209 + count)
    n = len(WIDTHS)
    g = mtgp.Generators(p, seeds)
    states = np.stack([oracle.seed(int(s), N) for s in seeds])
    counts = [count - (k % 3) for k in range(n)]
    dts = [k & 1 for k in range(n)]
    outs = [torch.empty(c, dtype=torch.int32, device="cuda") for c in counts]
    items = [(k, dts[k], counts[k], outs[k]) for k in range(n)]
    ws = g.workspace(items)
    for _ in range(2):
        g.batch(items, ws)
        for k in range(n):
            e, states[k] = oracle.generate(p[k], states[k], counts[k], as_float=bool(dts[k]))
            got = outs[k].cpu().numpy().view(np.uint32)
            assert np.array_equal(got, np.asarray(e).view(np.uint32)), WIDTHS[k]
        assert np.array_equal(g.states_host(), states)
        assert mtgp.batch_errors(ws) == 0
    # too little room for groups: fewer splits, the same numbers
    small = torch.empty(max(mtgp.batch_workspace_bytes(n), ws.numel() // 3 // 256 * 256),
                        dtype=torch.uint8, device="cuda")
    g.batch(items, small)
    for k in range(n):
        e, states[k] = oracle.generate(p[k], states[k], counts[k], as_float=bool(dts[k]))
        assert np.array_equal(outs[k].cpu().numpy().view(np.uint32), np.asarray(e).view(np.uint32))
    assert np.array_equal(g.states_host(), states)
    g.close()


def test_repairs_among_many_requests(torch):
    """More requests than waves check one each: foreign states written behind
    the library's back are found and regenerated wherever they lie."""
    n, count = 2600, 33000
    p = workloads.make_params(3217, n, 0x6E9A)
    p[:, 1] = N - 2 - (np.arange(n) % 30)          # W = 2 .. 31
    seeds = np.arange(1, n + 1, dtype=np.uint32)
    g = mtgp.Generators(p, seeds)
    out = torch.empty(n * count, dtype=torch.int32, device="cuda")
    items = [(k, mtgp.U32, count, out.data_ptr() + 4 * k * count) for k in range(n)]
    ws = g.workspace(items)
    bad = [0, 1, 63, 1300, 1301, n - 1]
    rows = g.states_host()
    rng = np.random.default_rng(4)
    for k in bad:
        rows[k] = rng.integers(0, 1 << 32, N, dtype=np.uint32)
    g.d_states.copy_(torch.from_numpy(rows.view(np.int32).reshape(-1)))
    g.batch(items, ws)
    got = out.cpu().numpy().view(np.uint32).reshape(n, count)
    after = g.states_host()
    repaired = mtgp.batch_errors(ws)
    print("case many repairs: %d" % repaired, flush=True)
    assert repaired <= len(bad)
    for k in bad + [2, 64, 700, 2048, n - 2]:
        e, st = oracle.generate(p[k], rows[k], count)
        assert np.array_equal(got[k], e), k
        assert np.array_equal(after[k], st), k
    g.close()
