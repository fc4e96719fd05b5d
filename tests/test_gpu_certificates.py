"""GPU tests of the edge-disjoint subgraphs' test and the threshold bound:
whole solves, single and batched, against the CPU oracle, at the sizes where
the kernels' tiles, unit counts and classes have their edges.

The graphs are two random blocks whose cheapest separation is one unit below
the smallest degree, so a union across it (a certificate that does not hold)
gives a wrong lambda, or it is above, so the answer is a single vertex."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2609_07204_amd as mc
    return mc.Context(0)


def two_blocks(n, degree, wmax, seed, bridge, hub=0):
    """Two random graphs of n // 2 and n - n // 2 vertices (a Hamiltonian
    cycle each, and random edges up to the mean degree), joined by edges of
    total weight (smallest degree inside) + bridge; hub: vertex 0 joined to
    that many vertices of its block by extra edges."""
    r = np.random.default_rng(seed)
    us, vs = [], []
    for lo, size in ((0, n // 2), (n // 2, n - n // 2)):
        p = lo + r.permutation(size)
        m = max(0, size * (degree - 2) // 2)
        us += [p, lo + r.integers(0, size, m)]
        vs += [np.roll(p, 1), lo + r.integers(0, size, m)]
    if hub:
        us.append(np.zeros(hub, np.int64))
        vs.append(1 + r.permutation(n // 2 - 1)[:hub])
    u, v = np.concatenate(us), np.concatenate(vs)
    w = r.integers(1, wmax + 1, u.size)
    g = gen.from_edges(n, u, v, w)
    deg = np.zeros(n, np.int64)
    np.add.at(deg, np.repeat(np.arange(n), np.diff(g.row_ptr)), g.w)
    left = int(deg.min()) + bridge
    u, v, w = g.edges()
    parts = min(max(left, 1), 7)
    cross = np.full(parts, max(left, 1) // parts, np.int64)
    cross[0] += max(left, 1) - cross.sum()
    u = np.concatenate([u, r.choice(n // 2, parts, replace=False)])
    v = np.concatenate([v, n // 2 + r.choice(n - n // 2, parts, replace=False)])
    return gen.from_edges(n, u, v, np.concatenate([w, cross]), "blocks(%d,%d,%d)" % (n, degree, wmax))


def check(ctx, g):
    lam_ref, _ = oracle.noi(g)
    lam, side, st = ctx.mincut(g, return_stats=True)
    assert lam == lam_ref, (g.name, lam, lam_ref, st)
    assert side[0] == 0 and 0 < side.sum() < g.n and oracle.cut_value(g, side) == lam
    return st


# n: just above the finisher's largest graph, multiples of the row tile and
# of the wavefront and one beside them; degree and wmax: fewer units than
# subgraphs, unit weights (k = lam below, at and above the largest k), units
# of weight 1 and of many, weights beyond 32 bits
@pytest.mark.parametrize("n,degree,wmax", [
    (1025, 24, 100), (1088, 30, 1), (1089, 40, 1), (1151, 80, 1), (2048, 16, 3), (2113, 31, 1000),
    (4097, 20, 1 << 40), (6000, 12, 10), (16385, 14, 100)])
@pytest.mark.parametrize("bridge", [-1, 5])
def test_solve_near_the_smallest_degree(ctx, n, degree, wmax, bridge):
    check(ctx, two_blocks(n, degree, wmax, n + degree, bridge))


# a row longer than the entries the test looks at, owned by the heaviest vertex
def test_long_row(ctx):
    check(ctx, two_blocks(12000, 10, 7, 5, -1, hub=5500))


def test_certificates_replace_capforest(ctx):
    # a sparse random graph with wide weights: no pass of CAPFOREST is needed
    g = gen.erdos_renyi(5000, 24 / 5000.0, 11, 1, 1000, lcc=True)
    st = check(ctx, g)
    assert st["marks_capforest"] == 0 and st["fallback_passes"] == 0
    # two communities: the threshold's parts give the bound at once
    g = gen.planted(3000, 3000, 16, 5, 1, 100, 3)
    st = check(ctx, g)
    assert st["marks_capforest"] == 0


def test_batch_mixes_graphs(ctx):
    # every kind in one batch, so the classes, references and thresholds of
    # neighbouring graphs meet inside one wavefront and one tile
    gs = []
    for i, (n, d, w) in enumerate([(1025, 24, 100), (70, 8, 5), (1500, 40, 1), (2113, 31, 1000), (1030, 12, 10),
                                   (3001, 16, 100), (64, 20, 1), (5000, 24, 1 << 33)]):
        gs.append(two_blocks(n, d, w, 100 + i, -1 if i % 2 else 4))
    gs.append(gen.planted(1200, 1300, 14, 5, 1, 100, 9))
    gs.append(gen.erdos_renyi(4000, 30 / 4000.0, 12, 1, 100, lcc=True))
    want = [oracle.noi(g)[0] for g in gs]
    for order in (range(len(gs)), reversed(range(len(gs)))):
        idx = list(order)
        lams, sides = ctx.mincut_batch([gs[i] for i in idx])
        for q, i in enumerate(idx):
            assert lams[q] == want[i], (gs[i].name, lams[q], want[i])
            assert sides[q][0] == 0 and oracle.cut_value(gs[i], sides[q]) == want[i]
