"""Plain calls on both sides of the line between the kernel for few streams
and the full chip's, every width of a narrow stream among them."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu

PER_CU = {3217: 6, 11213: 8, 23209: 16, 44497: 16}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("mexp", [3217, 11213, 23209, 44497])
def test_around_the_line(torch, mexp, over):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    N, n = mexp // 32 + 1, PER_CU[mexp] * cus + over
    print("case few streams mexp=%d n=%d" % (mexp, n), flush=True)
    p = workloads.make_params(mexp, n, 0xFE3)
    p[:62, 1] = N - 2 - np.arange(62)
    seeds = np.arange(n, dtype=np.uint32)
    g = mtgp.Generators(p, seeds)
    look = list(range(70)) + [n - 1]
    states = {k: oracle.seed(int(seeds[k]), N) for k in look}
    for count, dt in ((N + 3, 0), (1, 1), (601, 1)):
        got = g.generate(count, dt).cpu().numpy().view(np.uint32).reshape(n, count)
        for k in look:
            e, states[k] = oracle.generate(p[k], states[k], count, as_float=bool(dt))
            assert np.array_equal(got[k], np.asarray(e).view(np.uint32)), (count, k)
    after = g.states_host()
    for k in look:
        assert np.array_equal(after[k], states[k]), k
    g.close()
