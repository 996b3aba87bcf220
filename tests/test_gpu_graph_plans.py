"""Plans replayed from captured graphs on one workspace: two parameter sets
in the same buffers whose plans have the same numbers of items but other
table offsets must not share a graph."""
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


@pytest.mark.parametrize("mexp,count,widths", [(3217, 262144, (6, 12, 24, 6)),
                                               (11213, 1 << 20, (200, 160, 300, 200))])
def test_plans_of_one_workspace(torch, mexp, count, widths):
    n, N = 8, mexp // 32 + 1
    seeds = np.arange(1, n + 1, dtype=np.uint32)
    p = workloads.make_params(mexp, n, 0x6A9)
    out = torch.empty(n * count, dtype=torch.int32, device="cuda")
    items = [(k, mtgp.U32, count, out.data_ptr() + 4 * k * count) for k in range(n)]
    g = mtgp.Generators(p, seeds)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    for w in widths:
        print("case graph plans mexp=%d W=%d" % (mexp, w), flush=True)
        p[:, 1] = N - w
        mtgp.init_states(p, seeds, g.d_params, g.d_states, g.stride)
        states = np.stack([oracle.seed(int(s), N) for s in seeds])
        for _ in range(3):
            g.batch(items, ws)
            torch.cuda.synchronize()
            got = out.cpu().numpy().view(np.uint32).reshape(n, count)
            for k in range(n):
                e, states[k] = oracle.generate(p[k], states[k], count)
                assert np.array_equal(got[k], e), (w, k)
            assert np.array_equal(g.states_host(), states)
    assert mtgp.batch_errors(ws) == 0
    g.close()
