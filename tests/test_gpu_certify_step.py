"""GPU tests of the edge-disjoint subgraphs' test on its own
(mc_step_certify): every pair it joins is as connected as it claims, and the
trees it counts as joined are those that are gone, whatever forest it starts
from."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2609_07204_amd as mc
    return mc.Context(0)


def dev_of(ctx, g):
    return ctx.step_contract(ctx.dgraph(g))[0]


def sparse(n, degree, wmax, seed):
    r = np.random.default_rng(seed)
    p = r.permutation(n)
    m = n * (degree - 2) // 2
    u, v = np.concatenate([p, r.integers(0, n, m)]), np.concatenate([np.roll(p, 1), r.integers(0, n, m)])
    return gen.from_edges(n, u, v, r.integers(1, wmax + 1, u.size))


# every pair of small graphs against the minimum cut between the two
@pytest.mark.parametrize("seed", range(8))
def test_joined_pairs_are_connected(ctx, seed):
    g = gen.random_small(11 + seed % 4, 0.7, 900 + seed, 1, 9)
    dmin = int(oracle.degrees(g).min())
    dev = dev_of(ctx, g)
    joined = 0
    for lam in sorted({1, 2, max(1, dmin // 2), max(1, dmin), dmin + 5, 2 * dmin + 3}):
        lab, n2, marks = ctx.step_certify(dev, lam)
        assert marks == g.n - n2
        for x in range(g.n):
            for y in range(x + 1, g.n):
                if lab[x] == lab[y]:
                    joined += 1
                    assert oracle.brute_st(g, x, y) >= lam
    assert joined > 0


# a cut one unit below the bound keeps two blocks apart; the blocks join
@pytest.mark.parametrize("n,degree,wmax", [(1500, 24, 100), (4098, 30, 1), (40000, 20, 1000)])
def test_cut_below_the_bound(ctx, n, degree, wmax):
    h = n // 2
    a, b = sparse(h, degree, wmax, n), sparse(n - h, degree, wmax, n + 1)
    g = gen.disjoint_union(a, b)
    lam = int(oracle.degrees(g).min())
    u, v, w = g.edges()
    g = gen.from_edges(n, np.append(u, 3), np.append(v, h + 5), np.append(w, lam - 1))
    lab, n2, marks = ctx.step_certify(dev_of(ctx, g), lam)
    assert n2 < n and not set(lab[:h]) & set(lab[h:]) and marks == n - n2


# trees that other tests have joined: pairs (v, w) whose w comes to the joining
# launch early and v late, so that both want to hang v's tree at once
@pytest.mark.parametrize("n", [70, 3000, 300000, 700000])
@pytest.mark.parametrize("seed", [1, 2])
def test_trees_joined_are_counted_once(ctx, n, seed):
    g = sparse(n, 24, 100, n + seed)
    dev = dev_of(ctx, g)
    lam = int(oracle.degrees(g).min())
    r = np.random.default_rng(seed)
    start = np.arange(n)
    late = 1 << 18                       # one step of the launch's threads
    if n > late:
        w = late + r.permutation(min(n - late, late))[:200000]
        start[w] = late - 1 - r.integers(0, 60000, w.size)
    else:
        w = r.permutation(np.arange(1, n))[:n // 2]
        start[w] = (w * r.random(w.size)).astype(np.int64)
    # compressed or not, the forest's roots are what is counted
    roots = int((start == np.arange(n)).sum())
    for _ in range(10 if n > late else 2):
        lab, n2, marks = ctx.step_certify(dev, lam, start)
        assert (lab == lab[start]).all() and marks == roots - n2
    assert n2 <= roots
