"""GPU tests of the server's host memory: a request that it can never admit is
checked and refused without a copy, and polled requests leave no more than the
pool's 512 MB."""
import os

import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


def resident():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[1]) * os.sysconf("SC_PAGESIZE")


def big(n, nnz):
    """A long list of entries (not symmetric, which is not checked by default)."""
    rp = np.linspace(0, nnz, n + 1).astype(np.int32)
    return gen.Graph(n, rp, (np.arange(nnz) % n).astype(np.int32), np.ones(nnz, np.int64))


def test_too_large_a_request_is_not_copied():
    import paper_2609_07204_amd as mc
    ctx = mc.Context(0)
    srv = mc.Server(ctx, hbm_bytes=512 << 20, max_inflight=8, max_request_n=1024, max_request_nnz=1 << 16)
    g = big(5000, 1 << 24)                       # 200 MB
    bad = big(5000, 1 << 24)
    bad.col[-1] = 5000
    before = resident()
    for _ in range(2):
        with pytest.raises(mc.MincutError) as e:
            srv.submit(g)
        assert e.value.code == -4
        with pytest.raises(mc.MincutError) as e:
            srv.submit(bad)                      # what is wrong with it comes first
        assert e.value.code == -2
    assert resident() - before < 32 << 20
    t = srv.submit(gen.wheel(20))
    while srv.poll(t) is None:
        srv.step()
    srv.close()
    ctx.close()
