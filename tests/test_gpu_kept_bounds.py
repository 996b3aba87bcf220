"""Kept results of a replay whose destination is shorter than the result, or
ends with it: the first is refused and nothing is written, the second and the
replay's other results arrive."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu

SIZE = 1000    # bytes; an allocation takes whole pages, so 4 more stay in it


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


@pytest.mark.parametrize("words", [SIZE // 4, SIZE // 4 + 1])
def test_destination_of_one_allocation(torch, words):
    print("case kept bounds words=%d" % words, flush=True)
    hip = mtgp.lib()      # its HIP runtime
    p = workloads.make_params(11213, 2, 0xB0D5)
    g = mtgp.Generators(p, np.array([1, 2], dtype=np.uint32))
    other = torch.zeros(5000, dtype=torch.int32, device="cuda")
    dst, base, size = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_size_t()
    host = np.full(SIZE // 4, 0x5A5A5A5A, dtype=np.uint32)
    assert hip.hipMalloc(ctypes.byref(dst), ctypes.c_size_t(SIZE)) == 0
    try:
        assert hip.hipMemGetAddressRange(ctypes.byref(base), ctypes.byref(size), dst) == 0
        assert base.value == dst.value and size.value == SIZE
        assert hip.hipMemcpy(dst, host.ctypes.data_as(ctypes.c_void_p), ctypes.c_size_t(SIZE),
                             1) == 0
        srv = mtgp.Server(g, 256 << 20, inflight=2, workspace_bytes_per_batch=8 << 20)
        try:
            def replay():
                srv.replay(np.zeros(2, dtype=np.uint64), np.arange(2, dtype=np.int32),
                           np.array([words, 5000], dtype=np.uint64), np.zeros(2, dtype=np.int32),
                           keep=[dst.value, other.data_ptr()])
            if 4 * words > SIZE:
                with pytest.raises(mtgp.MTGPError):
                    replay()
            else:
                replay()
        finally:
            srv.close()
        assert hip.hipMemcpy(host.ctypes.data_as(ctypes.c_void_p), dst, ctypes.c_size_t(SIZE),
                             2) == 0
    finally:
        hip.hipFree(dst)
    if 4 * words > SIZE:
        assert (host == 0x5A5A5A5A).all()
    else:
        assert np.array_equal(host, oracle.generate(p[0], oracle.seed(1, 351), words)[0])
        assert np.array_equal(other.cpu().numpy().view(np.uint32),
                              oracle.generate(p[1], oracle.seed(2, 351), 5000)[0])
    g.close()
