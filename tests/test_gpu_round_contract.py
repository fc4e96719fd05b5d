"""GPU parity of the contraction as the rounds of a solve run it (symmetric
graphs whose longest row is known): the row of a group with half of all
entries taken from the others' column, groups with dense accumulators read
row by row. Every row, entry by entry, against the CPU oracle."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2609_07204_amd as mc
    return mc.Context(0)


def check(ctx, g, lab, n2):
    import torch
    src, _, _ = ctx.step_contract(ctx.dgraph(g))
    dst, dmin, darg = ctx.step_contract(src, torch.as_tensor(lab.astype(np.int32)).cuda(), n2, in_round=True)
    rp, col, w = oracle.contract(g, lab.astype(np.int32), n2)
    drp, dcol, dw, ddeg = dst.to_canonical()
    assert np.array_equal(drp, rp) and np.array_equal(dcol, col) and np.array_equal(dw, w)
    deg = np.zeros(n2, np.int64)
    np.add.at(deg, np.repeat(np.arange(n2), np.diff(rp)), w)
    assert np.array_equal(ddeg, deg)
    assert dmin == deg.min() and darg == int(np.argmin(deg))


def core_and_pendants(block, pendants, seed, tied=0.5):
    """A block of two random cycles and pendant vertices with one to three
    edges into it, a part of them also joined to the next pendant."""
    r = np.random.default_rng(seed)
    us, vs = [], []
    for _ in range(2):
        p = r.permutation(block)
        us.append(p)
        vs.append(np.roll(p, 1))
    k = r.integers(1, 4, pendants)
    us.append(np.repeat(block + np.arange(pendants), k))
    vs.append(r.integers(0, block, int(k.sum())))
    t = np.flatnonzero(r.random(max(pendants - 1, 0)) < tied)
    us.append(block + t)
    vs.append(block + t + 1)
    u, v = np.concatenate(us), np.concatenate(vs)
    return gen.from_edges(block + pendants, u, v, r.integers(1, 1 << 20, u.size), "core(%d)+%d" % (block, pendants))


# The giant group's row: a workgroup takes 32 groups a step and holds 1024 finds
# before it writes them out. Groups for less than a step, for one step of every
# workgroup (32 x 1024) and one group more, and for so many steps that finds
# are written out in between (1,015,808 groups are the most without).
@pytest.mark.parametrize("groups", [2, 31, 32, 33, 1000, 32768, 32769, 70001, 1015808, 1015809, 1100001])
def test_giant_row(ctx, groups):
    pendants = groups - 1
    block = 2500
    g = core_and_pendants(block, pendants, groups, min(0.5, 3000 / pendants))
    giant = (groups - 1) // 2                     # the block's label, in the middle of the others
    lab = np.empty(g.n, np.int32)
    lab[:block] = giant
    rest = np.arange(groups)
    lab[block:] = rest[rest != giant]
    rows = np.bincount(lab, weights=np.diff(g.row_ptr), minlength=groups)
    assert rows[giant] > 2048 and 2 * rows[giant] >= g.nnz
    check(ctx, g, lab, groups)


# other large groups beside: dense accumulators (at least a quarter of the group
# count; read row by row up to rows of 8192 entries, by tiles with a longer
# one), hash tables, and members merged by one workgroup
@pytest.mark.parametrize("sizes,small,hub", [
    ((6000, 900, 700, 40), 300, 0), ((3000, 3000, 3000, 2900), 700, 0), ((30000, 2300, 1200, 100, 5), 11000, 0),
    ((20000, 9000, 3000), 500, 8193), ((20000, 9000, 3000), 500, 8192), ((9000, 5000), 40000, 0), ((900,) * 30, 64, 0)])
def test_large_groups(ctx, sizes, small, hub):
    r = np.random.default_rng(sum(sizes) + small)
    n = sum(sizes) + small
    u, v = r.integers(0, n, 4 * n), r.integers(0, n, 4 * n)
    if hub:
        keep = (u != 0) & (v != 0)
        u = np.concatenate([u[keep], np.zeros(hub, np.int64)])
        v = np.concatenate([v[keep], 1 + r.permutation(n - 1)[:hub]])
    g = gen.from_edges(n, u, v, r.integers(1, 100, u.size), "groups%s" % (sizes,))
    assert not hub or np.diff(g.row_ptr).max() == hub
    check(ctx, g, np.repeat(np.arange(len(sizes) + small), list(sizes) + [1] * small), len(sizes) + small)


@pytest.mark.parametrize("seed,parts", [(1, 0.5), (2, 0.05), (3, 0.002), (4, 1.0)])
def test_random_labels(ctx, seed, parts):
    g = gen.chung_lu(20000, 2.5, 12.0, seed, 1, 50, kcore=0, lcc=False)
    n2 = max(1, int(g.n * parts))
    lab = np.random.default_rng(seed).integers(0, n2, g.n)
    lab[:n2] = np.arange(n2)
    check(ctx, g, lab, n2)
