"""GPU tests of the finisher's workgroup pass, its reduction tests and its
slab merge: whole solves of graphs of at most 1024 vertices against the CPU
oracle, at the sizes where threads, wavefronts, slabs and packed keys have
their edges."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2609_07204_amd as mc
    return mc.Context(0)


def sparse(n, degree, wmax, seed):
    """A Hamiltonian cycle and random edges up to the mean degree."""
    r = np.random.default_rng(seed)
    p = r.permutation(n)
    m = max(0, n * (degree - 2) // 2)
    u = np.concatenate([p, r.integers(0, n, m)])
    v = np.concatenate([np.roll(p, 1), r.integers(0, n, m)])
    w = r.integers(max(1, wmax // 2) if wmax > 1 << 40 else 1, wmax + 1, u.size)
    return gen.from_edges(n, u, v, w, "sparse(%d,%d,%d)" % (n, degree, wmax))


def check(ctx, g, lam_ref=None):
    lam_ref = oracle.noi(g)[0] if lam_ref is None else lam_ref
    lam, side, st = ctx.mincut(g, return_stats=True)
    assert lam == lam_ref, (g.name, lam, lam_ref, st)
    assert side[0] == 0 and 0 < side.sum() < g.n and oracle.cut_value(g, side) == lam


# n: one thread, wavefront and workgroup more or less; slabs of one, of many
# and of four groups; weights that leave keys small, wide, at and beyond the
# packed keys' limit (2^52), up to sums near 2^62
@pytest.mark.parametrize("n", [3, 4, 63, 64, 65, 127, 257, 511, 1023, 1024])
@pytest.mark.parametrize("degree,wmax", [(4, 1), (8, 9), (30, 1000), (12, None), (6, None)])
def test_sparse(ctx, n, degree, wmax):
    # None: the largest weights whose total stays below 2^62
    check(ctx, sparse(n, degree, wmax or (1 << 61) // (n * degree), 7 * n + degree))


# rows longer than the workgroup's wavefronts take at once; everything capped
# at once (unit weights) and popped one by one (weights far below the bound)
@pytest.mark.parametrize("n,wmax", [(1024, 1), (700, 50)])
def test_dense(ctx, n, wmax):
    u, v = np.triu_indices(n, 1)
    r = np.random.default_rng(n)
    g = gen.from_edges(n, u, v, r.integers(1, wmax + 1, u.size))
    deg = np.zeros(n, np.int64)
    np.add.at(deg, np.repeat(np.arange(n), np.diff(g.row_ptr)), g.w)
    check(ctx, g, int(deg.min()))    # a cut of k vertices crosses at least k (n - k) edges


def test_closed_forms(ctx):
    for g in (gen.cycle([3, 9, 4, 4, 7, 2, 8] * 146), gen.two_cliques(500, 520, 11, 3), gen.wheel(1000),
              gen.random_tree(900, 5), gen.planted(400, 600, 10, 5, 1, 1000, 3)):
        check(ctx, g)


def test_queues_agree(ctx):
    gs = [sparse(n, d, w, n) for n, d, w in ((900, 8, 100), (1000, 24, 1000), (300, 6, 3), (200, 12, 1 << 50))]
    gs.append(gen.planted(300, 340, 8, 5, 1, 10, 6))
    want = [oracle.noi(g)[0] for g in gs]
    try:
        for queue in (0, 1, 2):
            ctx.set_options(queue=queue)
            for g, lam in zip(gs, want):
                check(ctx, g, lam)
            lams, sides = ctx.mincut_batch(gs)
            assert list(lams) == want
            for g, lam, side in zip(gs, want, sides):
                assert side[0] == 0 and oracle.cut_value(g, side) == lam
    finally:
        ctx.set_options(queue=0)


def test_disconnected(ctx):
    g = gen.disjoint_union(sparse(400, 6, 9, 1), sparse(300, 6, 9, 2))
    h = gen.permute(g, 4)[0]
    lam, side = ctx.mincut(h)
    assert lam == 0 and side[0] == 0 and side.sum() in (300, 400) and oracle.cut_value(h, side) == 0
