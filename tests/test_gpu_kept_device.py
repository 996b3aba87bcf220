"""Kept results are copied on the server's GPU, whichever GPU is current in
the thread that replays."""
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


@pytest.mark.parametrize("current", [0, 1])
def test_replay_with_another_current_device(torch, current):
    if torch.cuda.device_count() <= current:
        pytest.skip("needs %d GPUs" % (current + 1))
    print("case kept device current=%d" % current, flush=True)
    count = 20000
    p = workloads.make_params(11213, 1, 0xDE7)
    with torch.cuda.device(0):
        g = mtgp.Generators(p, np.array([3], dtype=np.uint32))
        out = torch.zeros(count, dtype=torch.int32, device="cuda:0")
        srv = mtgp.Server(g, 256 << 20, inflight=2, workspace_bytes_per_batch=8 << 20)
    try:
        with torch.cuda.device(current):
            srv.replay(np.zeros(1, dtype=np.uint64), np.zeros(1, dtype=np.int32),
                       np.array([count], dtype=np.uint64), np.zeros(1, dtype=np.int32),
                       keep=[out.data_ptr()])
            assert torch.cuda.current_device() == current
    finally:
        srv.close()
    assert np.array_equal(out.cpu().numpy().view(np.uint32),
                          oracle.generate(p[0], oracle.seed(3, 351), count)[0])
    g.close()
