"""GPU tests of one CAPFOREST pass on its own in the two forms that solves run
on small graphs: the finisher's workgroup pass and the pass with its state in
LDS (mc_step_capforest). The scan is a permutation from its start, alpha is
the capacity of its prefix, the bound follows it, and the marks join vertices
at least as connected as the bound."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu

BATCH, LDS = 6, 7


@pytest.fixture(scope="module")
def ctx():
    import paper_2609_07204_amd as mc
    return mc.Context(0)


def sparse(n, degree, wmax, seed, wmin=1):
    r = np.random.default_rng(seed)
    p = r.permutation(n)
    m = max(0, n * (degree - 2) // 2)
    u, v = np.concatenate([p, r.integers(0, n, m)]), np.concatenate([np.roll(p, 1), r.integers(0, n, m)])
    return gen.from_edges(n, u, v, r.integers(wmin, wmax + 1, u.size))


def device(ctx, g):
    dev, dmin, _ = ctx.step_contract(ctx.dgraph(g))
    return dev, dmin


def check_scan(g, res, lam, start, complete=True):
    order = res["order"]
    assert order[0] == start and np.unique(order).size == order.size
    assert not complete or order.size == g.n
    if res["best_len"] > 0:
        side = np.zeros(g.n, np.uint8)
        side[order[:res["best_len"]]] = 1
        assert oracle.cut_value(g, side) == res["best_alpha"] and res["lam"] == min(lam, res["best_alpha"])


@pytest.mark.parametrize("mode", [BATCH, LDS])
@pytest.mark.parametrize("seed", range(6))
def test_marked_pairs_are_connected(ctx, mode, seed):
    g = gen.random_small(11 + seed % 4, 0.6, 700 + seed, 1, 9)
    dev, dmin = device(ctx, g)
    if dmin == 0:
        pytest.skip("an isolated vertex")
    for lam in (max(1, dmin // 2), dmin, dmin + 7):
        for start in (0, g.n - 1):
            res = ctx.step_capforest(dev, lam, start=start, mode=mode)
            check_scan(g, res, lam, start)
            thr = min(lam, res["best_alpha"])
            lab = res["labels"]
            for x in range(g.n):
                for y in range(x + 1, g.n):
                    if lab[x] == lab[y]:
                        assert oracle.brute_st(g, x, y) >= thr


# n: wavefronts, the workgroup, and (LDS) several vertices a thread; weights
# that leave most vertices capped at once, or popped one by one
@pytest.mark.parametrize("mode,n", [(BATCH, 63), (BATCH, 65), (BATCH, 513), (BATCH, 1024), (LDS, 64), (LDS, 1023),
                                    (LDS, 1025), (LDS, 2049), (LDS, 8193), (LDS, 16256)])
@pytest.mark.parametrize("degree,wmin,wmax", [(8, 1, 1), (16, 1, 1000), (6, 1 << 43, 1 << 44)])
def test_marks_keep_lambda(ctx, mode, n, degree, wmin, wmax):
    g = sparse(n, degree, wmax, n + degree, wmin)
    dev, dmin = device(ctx, g)
    true = oracle.noi(g)[0]
    for start in (0, n // 2, n - 1):
        res = ctx.step_capforest(dev, dmin, start=start, mode=mode)
        check_scan(g, res, dmin, start)
        thr = min(dmin, res["best_alpha"])
        assert thr >= true
        if thr > true and res["n2"] >= 2:
            h = gen.Graph(res["n2"], *oracle.contract(g, res["labels"], res["n2"]))
            assert oracle.noi(h)[0] == true
        elif thr > true:
            raise AssertionError("everything joined above lambda")


# truncated passes: one from a given start, many from hashed ones
@pytest.mark.parametrize("cap", [1, 5, 300])
def test_truncated_lds_passes(ctx, cap):
    g = sparse(3000, 10, 9, cap)
    dev, dmin = device(ctx, g)
    res = ctx.step_capforest(dev, dmin, start=7, mode=LDS, len_cap=cap)
    assert 1 <= res["order"].size <= cap
    check_scan(g, res, dmin, 7, complete=False)
    true = oracle.noi(g)[0]
    res = ctx.step_capforest(dev, dmin, start=-1, mode=LDS, passes=32, len_cap=cap)
    thr = min(dmin, res["best_alpha"])
    if thr > true:
        h = gen.Graph(res["n2"], *oracle.contract(g, res["labels"], res["n2"]))
        assert oracle.noi(h)[0] == true


def test_lds_pass_refuses_what_does_not_fit(ctx):
    import paper_2609_07204_amd as mc
    for n, lam in ((16257, 4), (100, 1 << 48)):
        dev, _ = device(ctx, sparse(n, 4, 3, 1))
        with pytest.raises(mc.MincutError) as e:
            ctx.step_capforest(dev, lam, mode=LDS)
        assert e.value.code == -1
