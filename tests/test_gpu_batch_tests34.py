"""GPU tests of the rule that switches reduction tests 3 and 4 off in the
batched and served forms: what they gain is held against the graphs that they
looked at, not against everything beside them, and a round in which they look
at none does not count."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


def ring(n, k, wmax, seed):
    """Vertices on a circle, each joined to the k next on either side."""
    r = np.random.default_rng(seed)
    i, p = np.arange(n), r.permutation(n)
    u, v = np.concatenate([i] * k), np.concatenate([(i + d) % n for d in range(1, k + 1)])
    return gen.from_edges(n, p[u], p[v], r.integers(1, wmax + 1, u.size))


def serve(srv, gs):
    ts = [srv.submit(g) for g in gs]
    res = {}
    while len(res) < len(ts):
        srv.step()
        for t in ts:
            r = srv.poll(t) if t not in res else None
            if r is not None:
                res[t] = r
    return [res[t] for t in ts]


def server(ctx):
    import paper_2609_07204_amd as mc
    return mc.Server(ctx, hbm_bytes=4 << 30, max_inflight=64, max_request_n=70000, max_request_nnz=1 << 21,
                     solo_min_n=1 << 17)


# before the ring: graphs that other tests halve, with a hundred times the
# vertices that tests 3 and 4 join in a smaller ring beside them; and two blocks
# whose bound the thresholds lower, which leaves no graph to look at
@pytest.mark.parametrize("kind", ["large", "lowered"])
def test_tests34_stay_on(kind):
    import paper_2609_07204_amd as mc
    g = ring(3000, 6, 2, 1)
    if kind == "large":
        before = [gen.erdos_renyi(60000, 16 / 60000.0, s, 1, 100, lcc=True) for s in (1, 2, 3)] + [ring(1100, 6, 2, 2)]
    else:
        before = [gen.planted(1200, 1300, 14, 5, 1, 100, 9)]
    lam = oracle.noi(g)[0]
    rounds = {}
    for name, first, options in (("on", [], {}), ("off", [], {"pr_tri_deg_cap": 0}), ("after", before, {})):
        ctx = mc.Context(0, **options)
        srv = server(ctx)
        for x, r in zip(first, serve(srv, first)):
            assert oracle.cut_value(x, r[1]) == r[0]
        r = serve(srv, [g])[0]
        assert r[0] == lam and oracle.cut_value(g, r[1]) == lam
        rounds[name] = r[2]["rounds"]
        srv.close()
        ctx.close()
    print(kind, rounds)
    assert 2 * rounds["on"] < rounds["off"], rounds       # the tests matter on this graph
    assert 2 * rounds["after"] < rounds["off"], rounds
