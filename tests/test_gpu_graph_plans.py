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


# 4,000 streams of W = 12, then 24: 8 and 4 segments each, in both plans 4,000
# jump blocks and 8,000 work items
@pytest.mark.parametrize("mexp,n,count,widths", [(3217, 8, 262144, (6, 12, 24, 6)),
                                                 (3217, 4000, 262144, (12, 24, 12)),
                                                 (11213, 8, 1 << 20, (200, 160, 300, 200))])
def test_plans_of_one_workspace(torch, mexp, n, count, widths):
    N = mexp // 32 + 1
    look = [0, 1, 2, n // 2, n - 3, n - 2, n - 1]
    seeds = np.arange(1, n + 1, dtype=np.uint32)
    p = workloads.make_params(mexp, n, 0x6A9)
    out = torch.empty(n * count, dtype=torch.int32, device="cuda")
    items = [(k, mtgp.U32, count, out.data_ptr() + 4 * k * count) for k in range(n)]
    g = mtgp.Generators(p, seeds)
    ws = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    for w in widths:
        print("case graph plans mexp=%d W=%d" % (mexp, w), flush=True)
        p[:, 1] = N - w
        mtgp.init_states(p, seeds, g.d_params, g.d_states, g.stride)
        states = {k: oracle.seed(int(seeds[k]), N) for k in look}
        for _ in range(3):
            g.batch(items, ws)
            torch.cuda.synchronize()
            after = g.states_host()
            for k in look:
                got = out[k * count:(k + 1) * count].cpu().numpy().view(np.uint32)
                e, states[k] = oracle.generate(p[k], states[k], count)
                assert np.array_equal(got, e), (w, k)
                assert np.array_equal(after[k], states[k]), (w, k)
    assert mtgp.batch_errors(ws) == 0
    g.close()
