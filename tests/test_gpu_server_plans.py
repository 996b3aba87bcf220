"""The server's batches share the chip and their streams' powers of x: none is
planned in groups, which the same request in a batch of its own is."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu

MODE_GROUP = 16


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


def _modes(words, stream):
    """Mode words of the work items of a stream that lie in a workspace: an
    item starts with its stream and its mode."""
    at = np.flatnonzero(words[:-1] == stream)
    return [int(words[i + 1]) for i in at if i >= 64 and words[i + 1] < 32]


def test_server_plans_no_groups(torch):
    print("case server plans", flush=True)
    n, k, count = 4400, 4321, 300000
    p = workloads.make_params(3217, n, 0x5E21)
    p[k, 1] = 101 - 20
    g = mtgp.Generators(p, np.arange(n, dtype=np.uint32))
    out = torch.empty(count, dtype=torch.int32, device="cuda")
    ws = g.workspace([(k, 0, count, out)])
    ws.zero_()
    g.batch([(k, 0, count, out)], ws)
    e, state = oracle.generate(p[k], oracle.seed(k, 101), count)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), e)
    modes = _modes(ws.cpu().numpy().view(np.uint32), k)
    assert any(m & MODE_GROUP for m in modes), modes
    size = 8 << 20
    srv = mtgp.Server(g, 64 << 20, inflight=1, workspace_bytes_per_batch=size)
    try:
        srv.pool.zero_()
        torch.cuda.synchronize()
        srv.replay(np.zeros(1, dtype=np.uint64), np.array([k], dtype=np.int32),
                   np.array([count], dtype=np.uint64), np.zeros(1, dtype=np.int32),
                   keep=[out.data_ptr()])
        modes = _modes(srv.pool[:size].cpu().numpy().view(np.uint32), k)
    finally:
        srv.close()
    assert len(modes) >= 3 and not any(m & MODE_GROUP for m in modes), modes
    e, state = oracle.generate(p[k], state, count)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), e)
    g.close()
