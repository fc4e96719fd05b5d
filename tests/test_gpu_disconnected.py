"""GPU tests of disconnected inputs: lambda 0 and the complement of vertex 0's
component as the side, told before any pass of CAPFOREST, and before any
round where the graph is small or resists the reduction tests, in every place
that decides it (the finisher, one workgroup, the general form, a coarse
graph)."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


def hypercube(k, lo):
    i = np.arange(1 << k)
    return (np.concatenate([lo + i] * k), np.concatenate([lo + (i ^ (1 << b)) for b in range(k)]))


def torus(a, b, lo):
    i = np.arange(a * b).reshape(a, b)
    return (lo + np.concatenate([i.ravel()] * 2), lo + np.concatenate([np.roll(i, 1, 0).ravel(), np.roll(i, 1, 1).ravel()]))


def sparse(n, degree, seed, lo):
    r = np.random.default_rng(seed)
    p = r.permutation(n)
    m = max(0, n * (degree - 2) // 2)
    return lo + np.concatenate([p, r.integers(0, n, m)]), lo + np.concatenate([np.roll(p, 1), r.integers(0, n, m)])


def side_by_side(parts, seed, wmax=1):
    """The components (functions of their first vertex, with their sizes) as
    one graph with shuffled numbers; component of every vertex."""
    us, vs, comp, lo = [], [], [], 0
    for k, (size, make) in enumerate(parts):
        u, v = make(lo)
        us.append(u)
        vs.append(v)
        comp.append(np.full(size, k))
        lo += size
    u, v, comp = np.concatenate(us), np.concatenate(vs), np.concatenate(comp)
    p = np.random.default_rng(seed).permutation(lo)
    inv = np.empty(lo, np.int64)
    inv[p] = np.arange(lo)
    g = gen.from_edges(lo, inv[u], inv[v], np.random.default_rng(seed).integers(1, wmax + 1, u.size))
    return g, comp[p]


def check(ctx, g, comp, rounds=None, **kw):
    lam, side, st = ctx.mincut(kw.get("host", g), dev=kw.get("dev"), return_stats=True)
    assert lam == 0 and np.array_equal(side, (comp != comp[0]).astype(np.uint8)), st
    assert st["marks_capforest"] == 0 and st["fallback_passes"] == 0, st
    if rounds is not None:
        assert st["rounds"] == rounds, st
    return st


def cubes(k):
    return [(1 << k, lambda lo: hypercube(k, lo))] * 2


# hard components (a hypercube's rounds contract little): no round is run. Sizes
# of the finisher, of one workgroup's components, both ends, and beyond
@pytest.mark.parametrize("parts", [
    cubes(1), cubes(3), cubes(9), cubes(10), cubes(11), cubes(13),
    [(512, lambda lo: hypercube(9, lo)), (513, lambda lo: sparse(513, 6, 1, lo))],
    [(2, lambda lo: sparse(2, 2, 1, lo)), (1020, lambda lo: sparse(1020, 3, 1, lo))],
    [(4, lambda lo: sparse(4, 3, 2, lo))] * 2000,
    [(6000, lambda lo: sparse(6000, 16, 3, lo)), (4, lambda lo: sparse(4, 3, 4, lo))]])
@pytest.mark.parametrize("options", [{}, {"heuristic_min_n": 0}, {"capforest_mode": 0}, {"finish_max_n": -1}])
def test_small(parts, options):
    import paper_2609_07204_amd as mc
    g, comp = side_by_side(parts, len(parts))
    ctx = mc.Context(0, **dict({"heuristic_min_n": 1 << 20}, **options))
    check(ctx, g, comp, rounds=0)
    check(ctx, g, comp, rounds=0, host=None, dev=ctx.upload(g))
    ctx.close()


# from the heuristic's size on: told before it where the input resists the tests
# (tori), on a contraction where it does not; far more components than
# workgroups; the largest looked at before the heuristic and one beyond
@pytest.mark.parametrize("parts,rounds", [
    ([(22500, lambda lo: torus(150, 150, lo))] * 2, 0),
    ([(65536, lambda lo: torus(256, 256, lo))] * 2, 0),
    ([(65536, lambda lo: torus(256, 256, lo)), (65792, lambda lo: torus(257, 256, lo))], None),
    ([(20000, lambda lo: sparse(20000, 16, 5, lo))] * 2, None),
    ([(100000, lambda lo: sparse(100000, 16, 6, lo)), (4, lambda lo: sparse(4, 3, 7, lo))], None),
    ([(4, lambda lo: sparse(4, 3, 8, lo))] * 40000, None)])
@pytest.mark.parametrize("wmax", [1, 100])
def test_large(parts, rounds, wmax):
    import paper_2609_07204_amd as mc
    g, comp = side_by_side(parts, 3, wmax)
    for options in ({}, {"heuristic_min_n": 0}, {"capforest_mode": 0}):
        ctx = mc.Context(0, **options)
        check(ctx, g, comp, rounds if wmax == 1 and options.get("heuristic_min_n") is None else None)
        ctx.close()


# an input that is folded first: edges of weight zero join nothing
@pytest.mark.parametrize("n", [40, 900, 3000, 9000, 40000])
def test_zero_weights_do_not_connect(n):
    import paper_2609_07204_amd as mc
    r = np.random.default_rng(n)
    us, vs = [], []
    for k in range(2):
        u, v = sparse(n // 2, 6, n + k, k * (n // 2))
        us.append(u)
        vs.append(v)
    b = r.integers(0, n // 2, n)
    u = np.concatenate(us + [b])
    v = np.concatenate(vs + [n // 2 + r.integers(0, n // 2, n)])
    w = np.concatenate([np.ones(u.size - n, np.int64), np.zeros(n, np.int64)])
    keep = u != v
    g = gen.raw_csr(n, u[keep], v[keep], w[keep])
    comp = np.arange(n) // (n // 2)
    ctx = mc.Context(0)
    check(ctx, g, comp)
    check(ctx, g, comp, host=None, dev=ctx.upload(g))
    w[-1] = 1                                        # one edge across: connected
    h = gen.raw_csr(n, u[keep], v[keep], w[keep])
    assert ctx.mincut(h)[0] == 1
    ctx.close()


# connected inputs of the same sizes are not taken for disconnected ones: a path
# through shuffled numbers (the first entries of its rows join little at once)
@pytest.mark.parametrize("n", [3, 1000, 1024, 1025, 16383, 16384, 16385, 50000])
@pytest.mark.parametrize("heuristic", [0, 10000])
def test_paths_are_connected(n, heuristic):
    import paper_2609_07204_amd as mc
    p = np.random.default_rng(n).permutation(n)
    hub = np.arange(1, n, max(1, n // 40))           # and a vertex whose row is long
    u = np.concatenate([p[:-1], np.zeros(hub.size, np.int64)])
    v = np.concatenate([p[1:], hub])
    g = gen.from_edges(n, u, v, np.full(u.size, 5))
    ctx = mc.Context(0, heuristic_min_n=heuristic)
    lam, side, st = ctx.mincut(g, return_stats=True)
    assert lam > 0 and oracle.cut_value(g, side) == lam and lam == int(oracle.noi(g)[0])
    ctx.close()
