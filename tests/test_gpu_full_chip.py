"""The kernels of a full chip under the default tuning: plain calls of more
streams, and batches of more items, than the kernels for a nearly empty chip
take, with narrow streams of every kind among them; and whole requests that
run beside the jumps, told by the claims they leave in the workspace."""
from __future__ import annotations

import os

import numpy as np
import pytest

import oracle
from paper_1501_07701_amd import mtgp, workloads

pytestmark = pytest.mark.gpu

WHOLE_CLAIMS, WIDE_CLAIMS = 24, 25     # header words: claim counters


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    mtgp.lib()
    return t


def _header(ws):
    return ws[:256].cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("mexp", [11213, 23209, 44497])
def test_every_narrow_width(torch, mexp):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    N, n = mexp // 32 + 1, 16 * cus + 7
    print("case full chip mexp=%d n=%d" % (mexp, n), flush=True)
    p = workloads.make_params(mexp, n, 0xF011)
    # the streams that are looked at: W = 2 .. 64, some with sh2 = 0 or 31,
    # then some whose tables are not linear
    look = list(range(0, 63)) + list(range(70, 90)) + [n - 1]
    p[:63, 1] = N - 2 - np.arange(63)
    p[0:63:7, 3], p[3:63:9, 3] = 0, 31
    p[70:90, 1] = N - np.array([2, 3, 7, 15, 16, 17, 30, 31, 32, 33, 47, 48, 49, 55, 56, 57, 60, 62,
                                63, 64])
    p[70:90, 5:21] = (workloads.splitmix64(np.arange(320, dtype=np.uint64), 0xF012)
                      >> np.uint64(32)).astype(np.uint32).reshape(20, 16)
    seeds = np.arange(n, dtype=np.uint32)
    g = mtgp.Generators(p, seeds)
    states = {k: oracle.seed(int(seeds[k]), N) for k in look}
    most = N + 131
    out = torch.empty(n * most, dtype=torch.int32, device="cuda")
    ws = torch.zeros(mtgp.batch_workspace_bytes(n), dtype=torch.uint8, device="cuda")

    def compare(got, count, dt):
        for k in look:
            c = count(k)
            e, states[k] = oracle.generate(p[k], states[k], c, as_float=bool(dt))
            assert np.array_equal(got[k][:c], np.asarray(e).view(np.uint32)), (k, c)

    for c, dt in ((1, 1), (N + 130, 0), (517, 1)):
        got = g.generate(c, dt).cpu().numpy().view(np.uint32).reshape(n, c)
        compare(got, lambda k: c, dt)
        items = [(k, dt, 1 + (c + 31 * k) % most, out.data_ptr() + 4 * k * most) for k in range(n)]
        g.batch(items, ws)
        assert _header(ws)[WIDE_CLAIMS] == 0             # not planned as sparse
        got = out.cpu().numpy().view(np.uint32).reshape(n, most)
        compare(got, lambda k: 1 + (c + 31 * k) % most, dt)
    after = g.states_host()
    for k in look:
        assert np.array_equal(after[k], states[k]), k
    g.close()


@pytest.mark.parametrize("overlap", ["0", "default"])
@pytest.mark.parametrize("mexp,n_short", [(3217, 26), (11213, 0)])
def test_whole_requests_do_run_beside_the_jumps(torch, mexp, n_short, overlap):
    """At mexp 11213 with more items than a sparse batch has."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n_short = n_short or 6 * cus + 50
    N, n_long = mexp // 32 + 1, 10
    print("case beside the jumps mexp=%d overlap=%s" % (mexp, overlap), flush=True)
    n = n_long + n_short
    p = workloads.make_params(mexp, n, 0x0E72)
    p[0, 1] = N - 2
    seeds = np.arange(1, n + 1, dtype=np.uint32)
    counts = [400000 + 1111 * k for k in range(n_long)] + [150 + k % 97 for k in range(n_short)]
    look = list(range(n_long + 20)) + [n - 1]
    old, before = os.environ.get("MTGP_OVERLAP"), mtgp.get_tuning(mexp)
    if overlap == "0":
        os.environ["MTGP_OVERLAP"] = "0"
    else:
        os.environ.pop("MTGP_OVERLAP", None)
    try:
        t = before.as_tuple()
        mtgp.set_tuning(mexp, t[0], t[1], t[2], 256, t[4])
        g = mtgp.Generators(p, seeds)
        outs = [torch.empty(c, dtype=torch.int32, device="cuda") for c in counts]
        items = [(k, k % 2, counts[k], outs[k]) for k in range(n)]
        ws = g.workspace(items)
        states = {k: oracle.seed(int(seeds[k]), N) for k in look}
        for rep in range(3):
            g.batch(items, ws)
            hdr = _header(ws)
            assert (hdr[WHOLE_CLAIMS] > 0) == (overlap != "0")
            assert hdr[WIDE_CLAIMS] == 0
            for k in look:
                o, states[k] = oracle.generate(p[k], states[k], counts[k], bool(k % 2))
                got = outs[k].cpu().numpy().view(np.uint32)
                assert np.array_equal(got, np.asarray(o).view(np.uint32)), (rep, k)
        assert mtgp.batch_errors(ws) == 0
        after = g.states_host()
        for k in look:
            assert np.array_equal(after[k], states[k]), k
        g.close()
    finally:
        mtgp.set_tuning(mexp, *before.as_tuple())
        if old is None:
            os.environ.pop("MTGP_OVERLAP", None)
        else:
            os.environ["MTGP_OVERLAP"] = old
