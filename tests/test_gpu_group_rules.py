"""When narrow streams are cut into groups: not below the tuning's floor of
dependent steps, and down to the shortest requests where the floor is low,
with outputs, states and continuations against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu

MEXP, N = 3217, 101
WIDTHS = [2, 3, 4, 5, 7, 8, 9, 12, 16, 17, 25, 32, 33, 40, 50, 63, 64]


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


class _Floor:
    def __init__(self, floor):
        self.floor = floor

    def __enter__(self):
        self.before = mtgp.get_tuning(MEXP)
        t = self.before.as_tuple()
        mtgp.set_tuning(MEXP, t[0], t[1], t[2], self.floor, t[4])

    def __exit__(self, *exc):
        mtgp.set_tuning(MEXP, *self.before.as_tuple())


def _run(torch, counts, floor, split):
    n = len(WIDTHS)
    p = workloads.make_params(MEXP, n, 0x6A11)
    p[:, 1] = [N - w for w in WIDTHS]
    seeds = np.arange(5, n + 5, dtype=np.uint32)
    with _Floor(floor):
        g = mtgp.Generators(p, seeds)
        outs = [torch.empty(c, dtype=torch.int32, device="cuda") for c in counts]
        items = [(k, k & 1, counts[k], outs[k]) for k in range(n)]
        need = mtgp.batch_workspace_query(g.d_params, items)
        assert (need > mtgp.batch_workspace_bytes(n)) == split
        ws = g.workspace(items)
        states = [oracle.seed(int(s), N) for s in seeds]
        for _ in range(2):
            g.batch(items, ws)
            for k in range(n):
                e, states[k] = oracle.generate(p[k], states[k], counts[k], as_float=bool(k & 1))
                got = outs[k].cpu().numpy().view(np.uint32)
                assert np.array_equal(got, np.asarray(e).view(np.uint32)), WIDTHS[k]
        assert np.array_equal(g.states_host(), np.array(states))
        assert mtgp.batch_errors(ws) == 0
        g.close()


@pytest.mark.parametrize("count", [2 * 16384, 2 * 16384 + 7, 4 * 16384 - 1, 4 * 16384 + 1,
                                   8 * 16384, 8 * 16384 + 1, 150001])
def test_short_requests_in_groups(torch, count):
    print("case short groups count=%d" % count, flush=True)
    _run(torch, [count - (k % 2) * (k % 5) for k in range(len(WIDTHS))], 128, True)


def test_a_floor_that_was_set_stays(torch):
    """The tuning's least number of steps per segment holds for groups too:
    300,000 outputs are fewer than 8192 steps of any of these streams."""
    print("case group floor", flush=True)
    _run(torch, [300000 - 11 * k for k in range(len(WIDTHS))], 8192, False)


def test_repairs_among_many_split_requests(torch):
    """More split requests than waves check one each: foreign states written
    behind the library's back are found and regenerated wherever they lie."""
    n, count = 2600, 33000
    p = workloads.make_params(MEXP, n, 0x6E9A)
    p[:, 1] = N - 2 - (np.arange(n) % 30)          # W = 2 .. 31
    seeds = np.arange(1, n + 1, dtype=np.uint32)
    bad = [0, 1, 63, 1300, 1301, n - 1]
    with _Floor(128):
        g = mtgp.Generators(p, seeds)
        out = torch.empty(n * count, dtype=torch.int32, device="cuda")
        items = [(k, mtgp.U32, count, out.data_ptr() + 4 * k * count) for k in range(n)]
        ws = g.workspace(items)
        rows = g.states_host()
        rng = np.random.default_rng(4)
        for k in bad:
            rows[k] = rng.integers(0, 1 << 32, N, dtype=np.uint32)
        g.d_states.copy_(torch.from_numpy(rows.view(np.int32).reshape(-1)))
        g.batch(items, ws)
        got = out.cpu().numpy().view(np.uint32).reshape(n, count)
        after = g.states_host()
        repaired = mtgp.batch_errors(ws)
        print("case many split repairs: %d" % repaired, flush=True)
        # most random sets' seed orbits span less than the state space
        assert 1 <= repaired <= len(bad)
        for k in bad + [2, 64, 700, 2048, n - 2]:
            e, st = oracle.generate(p[k], rows[k], count)
            assert np.array_equal(got[k], e), k
            assert np.array_equal(after[k], st), k
        g.close()
