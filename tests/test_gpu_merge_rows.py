"""GPU tests of the row-wise kernels' edges: forests ranked and labelled by one
workgroup and by tiles, input rows on both sides of the length that takes a
workgroup of its own, and contractions whose large groups are read row by row,
left to the others' column (half of all entries), or looked up in a table."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2609_07204_amd as mc
    return mc.Context(0)


# one workgroup up to 4096 vertices, then tiles of 2048
@pytest.mark.parametrize("n", [1, 2, 63, 1025, 4095, 4096, 4097, 6143, 6144, 6145, 100003])
def test_labels(ctx, n):
    r = np.random.default_rng(n)
    m = n // 2
    a, b = r.integers(0, n, m).astype(np.int32), r.integers(0, n, m).astype(np.int32)
    ref, k = oracle.components(n, a, b)
    lab, n2 = ctx.step_components(n, a, b)
    assert n2 == k and np.array_equal(lab, ref)


def hubs(lengths, leaves, seed):
    """`leaves` vertices on three random Hamiltonian cycles (weights 20 to 50)
    and one hub per length, joined to that many of them; a hub's edges weigh 1,
    but for one of weight 40."""
    r = np.random.default_rng(seed)
    k = len(lengths)
    us, vs, ws = [], [], []
    for _ in range(3):
        p = k + r.permutation(leaves)
        us.append(p)
        vs.append(np.roll(p, 1))
        ws.append(r.integers(20, 51, leaves))
    for h, l in enumerate(lengths):
        us.append(np.full(l, h))
        vs.append(k + r.permutation(leaves)[:l])
        w = np.ones(l, np.int64)
        w[r.integers(0, l)] = 40
        ws.append(w)
    return gen.from_edges(k + leaves, np.concatenate(us), np.concatenate(vs), np.concatenate(ws), "hubs%s" % (lengths,))


# rows on both sides of 512 entries and of a workgroup's 2048 at a time; beside
# them what the input pass has to report of such a row: not normal, malformed,
# too heavy
@pytest.mark.parametrize("lengths", [(511, 512, 513), (300, 2047, 2048, 2049, 4097), (9000,), (600,) * 40])
@pytest.mark.parametrize("leaves", [4100, 12000])
def test_long_input_rows(ctx, lengths, leaves):
    import paper_2609_07204_amd as mc
    import torch
    if max(lengths) > leaves:
        pytest.skip("a hub longer than the cycles")
    g = hubs(lengths, leaves, leaves)
    lam_ref = oracle.noi(g)[0]
    rp, col, w = (np.array(x) for x in (g.row_ptr, g.col, g.w))

    def dev(col, w):
        return (torch.as_tensor(rp.astype(np.int32)).cuda(), torch.as_tensor(col.astype(np.int32)).cuda(),
                torch.as_tensor(w.astype(np.int64)).cuda())
    for a in (dict(g=g), dict(dev=dev(col, w))):
        lam, side = ctx.mincut(**a)
        assert lam == lam_ref and oracle.cut_value(g, side) == lam
    h = len(lengths) - 1                        # the last hub's row
    last = int(rp[h + 1]) - 1
    swapped = col.copy()
    swapped[[last - 1, last]] = swapped[[last, last - 1]]
    ww = w.copy()
    ww[[last - 1, last]] = ww[[last, last - 1]]
    lam, side, st = ctx.mincut(dev=dev(swapped, ww), return_stats=True)
    assert lam == lam_ref and oracle.cut_value(g, side) == lam and st["input_normal"] == 0
    for c2, w2 in ((np.where(np.arange(col.size) == last, g.n, col), w),
                   (col, np.where(np.arange(col.size) == last, -1, w)),
                   (col, np.where(np.arange(col.size) == last, 1 << 62, w)),
                   (col, np.where((np.arange(col.size) == last) | (np.arange(col.size) == col.size - 1), 1 << 61, w))):
        with pytest.raises(mc.MincutError):
            ctx.mincut(dev=dev(c2, w2))
    assert ctx.mincut(dev=dev(col, w))[0] == lam_ref


# Blocks whose edges weigh more than a pendant vertex's degree, and pendant
# vertices that bound lambda: test 1 joins every block at once, so the first
# contraction has the blocks and the pendants as its groups. "giant": one block
# holds half of all entries; the others take accumulators (at least a quarter
# of the group count), a table (more than 2048 entries, fewer than that), or
# the merges for small and middle groups. A hub longer than 8192 entries keeps
# the tile path.
@pytest.mark.parametrize("blocks,pendants,hub", [
    ((6000, 900, 700, 40), 300, 0),             # giant, accumulators, middle
    ((2000, 2000, 2000, 1500), 3000, 0),        # accumulators only
    ((30000, 2300, 1200, 100, 5), 11000, 0),    # giant and a table
    ((3000, 2900, 10), 1, 0),
    ((20000, 9000, 3000), 500, 9000),           # a row of more than 8192 entries
    ((20000, 9000, 3000), 500, 8100),
])
def test_large_groups(ctx, blocks, pendants, hub):
    r = np.random.default_rng(sum(blocks) + pendants)
    us, vs, ws, lab, lo = [], [], [], [], 0
    for k, size in enumerate(blocks):
        for _ in range(2):
            p = lo + r.permutation(size)
            us.append(p)
            vs.append(np.roll(p, 1))
            ws.append(np.full(size, 1000))
        lab += [k] * size
        lo += size
    if hub:
        us.append(np.zeros(hub, np.int64))
        vs.append(1 + r.permutation(blocks[0] - 1)[:hub])
        ws.append(np.full(hub, 1000))
    m = 3 * pendants
    us.append(np.repeat(lo + np.arange(pendants), 3))
    vs.append(r.integers(0, lo, m))
    ws.append(r.integers(20, 60, m))
    lab += list(range(len(blocks), len(blocks) + pendants))
    # bridges between the blocks, a few
    b = 4 * len(blocks)
    us.append(r.integers(0, lo, b))
    vs.append(r.integers(0, lo, b))
    ws.append(r.integers(1, 30, b))
    n = lo + pendants
    g = gen.from_edges(n, np.concatenate(us), np.concatenate(vs), np.concatenate(ws), "blocks%s" % (blocks,))
    # no cut below 1000 divides a block, and a pendant vertex weighs less
    coarse = gen.Graph(len(blocks) + pendants, *oracle.contract(g, np.array(lab, np.int32), len(blocks) + pendants))
    lam_ref = oracle.noi(coarse)[0]
    assert lam_ref < 1000
    lam, side, st = ctx.mincut(g, return_stats=True)
    assert lam == lam_ref and oracle.cut_value(g, side) == lam, st
