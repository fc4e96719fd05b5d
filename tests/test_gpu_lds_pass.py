"""GPU tests of the CAPFOREST pass with its state in LDS (graphs of 1025 to
16,256 vertices, bounds below 2^48): whole solves with private passes asked for
by name, single and batched, against the CPU oracle, at the edges of its
sizes, its packed keys and its scan budget."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu

PRIVATE = 0    # MC_CF_PRIVATE


def sparse(n, degree, wmax, seed, wmin=1):
    r = np.random.default_rng(seed)
    p = r.permutation(n)
    m = max(0, n * (degree - 2) // 2)
    u = np.concatenate([p, r.integers(0, n, m)])
    v = np.concatenate([np.roll(p, 1), r.integers(0, n, m)])
    return gen.from_edges(n, u, v, r.integers(wmin, wmax + 1, u.size), "sparse(%d,%d,%d)" % (n, degree, wmax))


def check(ctx, g, lam_ref):
    lam, side, st = ctx.mincut(g, return_stats=True)
    assert lam == lam_ref, (g.name, lam, lam_ref, st)
    assert side[0] == 0 and 0 < side.sum() < g.n and oracle.cut_value(g, side) == lam
    return st


# n: the smallest and largest of the kernel, one beyond it (the pass in HBM),
# multiples of the workgroup and beside; weights that make keys small and large
@pytest.mark.parametrize("n", [1025, 2047, 2048, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("degree,wmin,wmax", [(6, 1, 1), (16, 1, 1000), (6, 1 << 44, 1 << 45)])
def test_private_solve(n, degree, wmin, wmax):
    import paper_2609_07204_amd as mc
    g = sparse(n, degree, wmax, n + degree, wmin)
    ctx = mc.Context(0, capforest_mode=PRIVATE, capforest_passes=3, heuristic_min_n=0, finish_max_n=-1,
                     pr_tri_deg_cap=0)
    st = check(ctx, g, oracle.noi(g)[0])
    assert st["rounds"] >= 1
    ctx.close()


# the largest graphs of the kernel: keys of 14 bits of vertex, all of the LDS
@pytest.mark.parametrize("n", [9000, 16255, 16256, 16257])
def test_largest_graphs(n):
    import paper_2609_07204_amd as mc
    for w in ((1, 1), (1 << 43, 1 << 44)):
        g = sparse(n, 6, w[1], n, w[0])
        ctx = mc.Context(0, capforest_mode=PRIVATE, capforest_passes=3, heuristic_min_n=0, finish_max_n=-1,
                         pr_tri_deg_cap=0)
        check(ctx, g, oracle.noi(g)[0])
        ctx.close()


# bounds of 2^49 and more, too large to be packed beside a vertex (the pass in
# HBM), on a cycle, whose minimum cut is its two lightest edges
def test_large_bounds():
    import paper_2609_07204_amd as mc
    ctx = mc.Context(0, capforest_mode=PRIVATE, heuristic_min_n=0, finish_max_n=-1)
    r = np.random.default_rng(1)
    for n in (1025, 1900):
        w = r.integers(1 << 49, 1 << 50, n)
        check(ctx, gen.permute(gen.cycle(w), n)[0], int(np.sort(w)[:2].sum()))
    ctx.close()


# truncated passes: a batch cut at the budget, and passes of one scan
@pytest.mark.parametrize("cap", [1, 7, 100])
def test_scan_budget(cap):
    import paper_2609_07204_amd as mc
    ctx = mc.Context(0, capforest_mode=PRIVATE, pass_len_cap=cap, heuristic_min_n=0, finish_max_n=-1)
    g = sparse(1500, 10, 5, cap)
    check(ctx, g, oracle.noi(g)[0])
    ctx.close()


def test_batch_of_both_kinds():
    import paper_2609_07204_amd as mc
    gs = [sparse(n, d, w, n) for n, d, w in ((1100, 6, 9), (8192, 8, 50), (9000, 8, 50), (1025, 30, 1000), (3000, 5, 1))]
    gs.append(gen.planted(900, 1200, 12, 5, 1, 10, 2))
    want = [oracle.noi(g)[0] for g in gs]
    ctx = mc.Context(0, capforest_mode=PRIVATE, batch_lp=2)
    lams, sides = ctx.mincut_batch(gs)
    assert list(lams) == want
    for g, lam, side in zip(gs, want, sides):
        assert side[0] == 0 and oracle.cut_value(g, side) == lam
    ctx.close()
