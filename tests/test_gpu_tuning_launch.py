"""A launch that the caller chose is the one that runs, also where the chip is
nearly empty; the default one leaves the choice to the library.  Narrow
streams, non-linear tables and both types through every one-wave launch, in
plain calls and batches, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu

WIDE_CLAIMS = 25     # header word: items that whole workgroups claimed


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


@pytest.mark.parametrize("mexp", [11213, 23209, 44497])
def test_chosen_launches_run(torch, mexp):
    N = mexp // 32 + 1
    widths = [2, 3, 9, 17, 31, 32, 40, 63, 64, 127, 128, 256, N - 1, 5, 200]
    n = len(widths)
    p = workloads.make_params(mexp, n, 0x7A0E)
    p[:, 1] = [N - w for w in widths]
    p[3, 3] = 0                                           # sh2 = 0
    p[-2:, 5:21] = (workloads.splitmix64(np.arange(32, dtype=np.uint64), 0x7A0F)
                    >> np.uint64(32)).astype(np.uint32).reshape(2, 16)   # not linear
    seeds = np.arange(1, n + 1, dtype=np.uint32)
    calls = [(1, 0), (3 * N + 5, 1), (2003, 0)]
    before = mtgp.get_tuning(mexp)
    try:
        for cand in mtgp.tuning_candidates(mexp):
            if cand.threads_per_stream != 64:
                continue
            print("case launch mexp=%d" % mexp, cand.as_tuple(), flush=True)
            mtgp.set_tuning(mexp, *cand.as_tuple())
            g = mtgp.Generators(p, seeds)
            states = [oracle.seed(int(s), N) for s in seeds]
            out = [torch.empty(3 * N + 2003, dtype=torch.int32, device="cuda") for _ in range(n)]
            ws = torch.zeros(mtgp.batch_workspace_bytes(n), dtype=torch.uint8, device="cuda")
            for c, dt in calls:
                got = g.generate(c, dt).cpu().numpy().view(np.uint32).reshape(n, c)
                g.batch([(k, dt, c + k, out[k]) for k in range(n)], ws)
                claimed = int(ws[:256].cpu().numpy().view(np.uint32)[WIDE_CLAIMS])
                assert (claimed > 0) == (cand.as_tuple()[:3] == before.as_tuple()[:3])
                for k in range(n):
                    e, states[k] = oracle.generate(p[k], states[k], c, as_float=bool(dt))
                    assert np.array_equal(got[k], np.asarray(e).view(np.uint32)), widths[k]
                    e, states[k] = oracle.generate(p[k], states[k], c + k, as_float=bool(dt))
                    b = out[k][:c + k].cpu().numpy().view(np.uint32)
                    assert np.array_equal(b, np.asarray(e).view(np.uint32)), widths[k]
            assert np.array_equal(g.states_host(), np.array(states))
            g.close()
    finally:
        mtgp.set_tuning(mexp, *before.as_tuple())
