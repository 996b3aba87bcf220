"""The draw API's window of narrow streams at its edges, against the oracle:
step widths with one chunk, a few and many chunks per class, draws shorter
and longer than a window, shifts that keep or drop the carry, and a
recursion table that is not linear (steps instead)."""
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


@pytest.mark.parametrize("mexp", workloads.SUPPORTED_MEXP)
@pytest.mark.parametrize("threads", [64, 320, 1024])
def test_draws_of_narrow_streams(torch, mexp, threads):
    print("case window draws mexp=%d threads=%d" % (mexp, threads), flush=True)
    N = mexp // 32 + 1
    widths = [2, 3, 5, 7, 15, 16, 17, 21, 22, 31, 32, 33, 47, 62, 63, 64, 2, 9]
    p = workloads.make_params(mexp, len(widths), 0xD31 + threads)
    p[:, 1] = [N - w for w in widths]
    p[0, 3], p[1, 3], p[4, 3] = 0, 31, 1
    p[16:, 5:21] = (workloads.splitmix64(np.arange(32, dtype=np.uint64), 0xABC)
                    >> np.uint64(32)).astype(np.uint32).reshape(2, 16)   # not linear
    n = len(widths)
    seeds = np.arange(n, dtype=np.uint32)
    g = mtgp.Generators(p, seeds)
    states = np.stack([oracle.seed(int(s), N) for s in seeds])
    for c, dt in [(threads, mtgp.U32), (1, mtgp.F32), (threads + 2, mtgp.F32),
                  (7 * threads + 63, mtgp.U32)]:
        out = torch.empty(n * c, dtype=torch.int32, device="cuda")
        mtgp.generate_workgroup(g.d_params, g.d_states, g.stride, n, c, out, dt, threads)
        got = out.cpu().numpy().view(np.uint32).reshape(n, c)
        exp, states = oracle.generate_many(p, states, c, dt == mtgp.F32, threads=8)
        for k in range(n):
            assert np.array_equal(got[k], np.asarray(exp[k]).view(np.uint32)), (c, dt, widths[k])
    assert np.array_equal(g.states_host(), states)
    g.close()
