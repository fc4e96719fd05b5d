"""Performance cases of the exact minimum-cut solver.

Every case is work that a program gives this library through its Python
entry points: one exact solve of a graph in device or host memory
(Context.mincut), a batch of graphs solved in one call
(Context.mincut_batch), or a set of requests answered by the server (Server).
The graph families and their parameters are those of the repository's
generators and benchmark (planted, Erdos-Renyi, Chung-Lu, cores of Chung-Lu
and of random hyperbolic graphs), generated here on the GPU from a seed.

A case is a dict of plain values:
  kind       "solve", "batch" or "serve"
  family     planted | er | chung_lu | hyperbolic (solve)
  n, degree  vertices and mean degree before the core is taken (solve)
  core       0, or k: the largest component of the k-core (solve); of these
             the value and the input's sizes are asked for, as the benchmark
             does, of all others the value and a side
  wmax       weights are uniform in [1, wmax]
  host       the graph is in host memory (solve, batch)
  raw        rows unsorted, with loops and parallel entries (solve)
  heuristic  False: the label-propagation bound is switched off (solve)
  count, nmin, nmax        graphs and their sizes, log-uniform (batch)
  count, mmin, mmax        requests and their edges, log-uniform (serve)
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2609_07204_amd as mc


def _solve(name, family, n, degree, wmax, core=0, host=False, raw=False, heuristic=True):
    c = {"kind": "solve", "family": family, "n": n, "degree": degree, "wmax": wmax, "core": core, "host": host,
         "raw": raw, "heuristic": heuristic}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a small graph handed over as numpy arrays, as a program that solves
        # one cluster or one partition at a time does: latency only
        _solve("planted_128_host", "planted", 128, 8, 10, host=True),
        # two regular communities joined by five light edges, resident on the
        # GPU (the benchmark's planted configuration)
        _solve("planted_2000", "planted", 2000, 12, 10),
        # an ordinary request: a sparse random graph from host memory
        _solve("er_16k_host", "er", 16384, 16, 100, host=True),
        # an ordinary power-law graph with wide weights, odd size, resident
        _solve("chung_lu_60k", "chung_lu", 60001, 20, 1000),
        # an edge list as it was collected: unsorted rows, loops and parallel
        # entries that the solver folds first
        _solve("er_200k_raw", "er", 200003, 16, 100, raw=True),
        # the served pool's heavy kind: millions of edges, weights to 1000
        _solve("er_300k", "er", 300000, 24, 1000),
        # cores of power-law graphs with unit weights (network reliability of
        # a social or web graph), a moderate and a large one
        _solve("chung_lu_2e20_core10", "chung_lu", 1 << 20, 20, 1, core=10),
        _solve("chung_lu_2e22_core10", "chung_lu", 1 << 22, 20, 1, core=10),
        # the 32-core of a random hyperbolic graph, the family of the
        # benchmark's headline; the largest single solve
        _solve("hyperbolic_2e21_core32", "hyperbolic", 1 << 21, 64, 100, core=32),
        # the same family with the bound heuristic off: many rounds of
        # reduction tests, CAPFOREST passes and contractions at full size
        _solve("hyperbolic_2e20_rounds", "hyperbolic", 1 << 20, 64, 100, core=32, heuristic=False),
        # many graphs of mixed families and sizes in one call (the
        # benchmark's batch, fewer of them)
        {"name": "batch_384", "kind": "batch", "count": 384, "nmin": 64, "nmax": 65536, "wmax": 100, "host": False},
        # a queue of requests of mixed families and sizes answered by the
        # server (host graphs, as it takes them)
        {"name": "serve_32", "kind": "serve", "count": 32, "mmin": 1000, "mmax": 3000000, "wmax": 1000},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges; none costs more than the largest
    listed single solve, batch or set of requests."""
    kind = rng.choice(["solve"] * 8 + ["batch", "serve"])
    if kind == "batch":
        return {"kind": "batch", "count": _log_uniform(rng, 8, 256), "nmin": 64,
                "nmax": _log_uniform(rng, 2048, 65536), "wmax": 100, "host": rng.random() < 0.5}
    if kind == "serve":
        return {"kind": "serve", "count": rng.randint(4, 24), "mmin": 1000,
                "mmax": _log_uniform(rng, 30000, 2000000), "wmax": 1000}
    family = rng.choice(["planted", "er", "chung_lu", "core", "hyperbolic"])
    degree, wmax = rng.randint(8, 32), rng.choice([10, 100, 1000])
    if family == "core":
        return _solve(None, "chung_lu", _log_uniform(rng, 1 << 14, 1 << 21), 20, 1, core=10)
    if family == "hyperbolic":
        return _solve(None, "hyperbolic", _log_uniform(rng, 1 << 14, 1 << 20), 64, 100, core=32,
                      heuristic=rng.random() < 0.75)
    n = _log_uniform(rng, 128, 1000000 if family == "planted" else 200000)
    host = n < 100000 and rng.random() < 0.4
    return _solve(None, family, n, degree, wmax, host=host, raw=not host and rng.random() < 0.2)


# ------------------------------------------------------------ generators
def _uniform(g, shape):
    return torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)


def _ints(g, lo, hi, size):
    return torch.randint(lo, hi, (size,), generator=g, device="cuda", dtype=torch.int64)


def _planted(n, d, g):
    """Two random, nearly d-regular blocks (d/2 random cycles each) joined by
    five edges; the last five edges returned are those."""
    us, vs = [], []
    for lo, size in ((0, n // 2), (n // 2, n - n // 2)):
        order = torch.argsort(_uniform(g, (max(1, d // 2), size)), dim=1)
        us.append((lo + order).reshape(-1))
        vs.append((lo + torch.roll(order, 1, 1)).reshape(-1))
    us.append(_ints(g, 0, n // 2, 5))
    vs.append(_ints(g, n // 2, n, 5))
    return torch.cat(us), torch.cat(vs)


def _er(n, d, g):
    return _ints(g, 0, n, n * d // 2), _ints(g, 0, n, n * d // 2)


def _chung_lu(n, d, g):
    """Expected degrees c (i+1)^(-1/1.5) (exponent 2.5) of mean d, capped at
    sqrt(n d)."""
    w = torch.arange(1, n + 1, device="cuda", dtype=torch.float64) ** (-1.0 / 1.5)
    cum = torch.cumsum(torch.clamp(w * (d * n / w.sum()), max=math.sqrt(n * d)), 0)
    m = int(cum[-1].item() / 2)
    return tuple(torch.searchsorted(cum, _uniform(g, (m,)) * cum[-1]).clamp_(max=n - 1) for _ in range(2))


def _hyperbolic(n, d, g):
    """Threshold random hyperbolic graph of exponent 5 (radial density
    parameter 2): points nearer than the disk radius are joined. Points are
    split into bands of the distance t from the rim; a pair of bands is
    searched over the widest angle that can join its points."""
    alpha = 2.0
    xi = alpha / (alpha - 0.5)
    radius = 2.0 * math.log(2.0 * xi * xi * n / (math.pi * d))
    t = radius - torch.acosh(1 + (math.cosh(alpha * radius) - 1) * _uniform(g, (n,))) / alpha
    theta = torch.sort(_uniform(g, (n,)) * (2 * math.pi))[0]
    width = 0.5
    band = (t / width).long()
    members = [torch.nonzero(band == b).view(-1) for b in range(int(band.max().item()) + 1)]
    us, vs = [], []
    for a, ia in enumerate(members):
        for b in range(a, len(members)):
            ib = members[b]
            if not ia.numel() or not ib.numel():
                continue
            reach = min(math.pi, 2.0 * math.exp(((a + b + 2) * width - radius) / 2))
            tb = theta[ib]
            turned = torch.cat([tb - 2 * math.pi, tb, tb + 2 * math.pi])
            lo = torch.searchsorted(turned, theta[ia] - reach)
            count = torch.searchsorted(turned, theta[ia] + reach) - lo
            first = torch.cumsum(count, 0) - count
            at = torch.repeat_interleave(torch.arange(ia.numel(), device="cuda"), count)
            j = torch.arange(at.numel(), device="cuda") - first[at] + lo[at]
            x, y = ia[at], ib[j % ib.numel()]
            gap = torch.remainder(theta[x] - theta[y], 2 * math.pi)
            near = torch.minimum(gap, 2 * math.pi - gap) <= 2.0 * torch.exp((t[x] + t[y] - radius) / 2)
            near &= (x < y) if a == b else (x != y)
            us.append(x[near])
            vs.append(y[near])
    return torch.cat(us), torch.cat(vs)


_FAMILY = {"planted": _planted, "er": _er, "chung_lu": _chung_lu, "hyperbolic": _hyperbolic}


def _components(n, u, v):
    """Smallest vertex of each vertex's component."""
    f = torch.arange(n, device="cuda")
    while True:
        a, b = f[u], f[v]
        low = torch.minimum(a, b)
        h = f.scatter_reduce(0, a, low, "amin").scatter_reduce_(0, b, low, "amin")
        while True:
            p = h[h]
            if torch.equal(p, h):
                break
            h = p
        if torch.equal(h, f):
            return f
        f = h


def _graphs(specs, wmax, g, raw=False):
    """Device graphs (row_ptr, col, w), one per spec (family, n, degree,
    core): the edges of all are drawn, made connected (the largest component
    of the core; without a core every other component is tied to the largest
    by one edge, so all n vertices stay), given shuffled vertex numbers and
    laid out as CSR together."""
    us, vs, ones, gid, n = [], [], [], [], 0
    for k, (family, size, d, _) in enumerate(specs):
        u, v = _FAMILY[family](size, d, g)
        us.append(u + n)
        vs.append(v + n)
        one = torch.zeros(u.numel(), dtype=torch.bool, device="cuda")
        if family == "planted":
            one[-5:] = True
        ones.append(one)
        gid.append(torch.full((size,), k, device="cuda"))
        n += size
    u, v, one, gid = torch.cat(us), torch.cat(vs), torch.cat(ones), torch.cat(gid)
    del us, vs, ones
    w = torch.where(one, 1, _ints(g, 1, wmax + 1, u.numel()))
    # simple graph: loops and repeated pairs dropped
    key, order = torch.sort(torch.minimum(u, v) * n + torch.maximum(u, v), stable=True)
    keep = torch.ones_like(one)
    keep[1:] = key[1:] != key[:-1]
    u, v, w = key // n, key % n, w[order]
    keep &= u != v
    u, v, w = u[keep], v[keep], w[keep]
    core = specs[0][3]
    while core:
        low = (torch.bincount(u, minlength=n) + torch.bincount(v, minlength=n)) < core
        keep = ~(low[u] | low[v])
        if bool(keep.all().item()):
            break
        u, v, w = u[keep], v[keep], w[keep]
    # largest component of each graph
    root = _components(n, u, v)
    size = torch.bincount(root, minlength=n)
    score = size * (n + 1) + (n - torch.arange(n, device="cuda"))
    best = torch.zeros(len(specs), dtype=torch.int64, device="cuda").scatter_reduce_(0, gid, score, "amax")
    best = (n - best % (n + 1))[gid]
    kept = best == root
    if not core:
        main, count = torch.nonzero(kept).view(-1), torch.bincount(gid[kept], minlength=len(specs))
        first = torch.cumsum(count, 0) - count
        tie = torch.nonzero((root == torch.arange(n, device="cuda")) & ~kept).view(-1)
        to = main[first[gid[tie]] + (_uniform(g, (tie.numel(),)) * count[gid[tie]]).long()]
        u, v, w = torch.cat([u, tie]), torch.cat([v, to]), torch.cat([w, _ints(g, 1, wmax + 1, tie.numel())])
        kept = torch.ones_like(kept)
    # shuffled numbers, graph by graph
    old = torch.nonzero(kept).view(-1)
    old = old[torch.argsort(gid[old] + _uniform(g, (old.numel(),)))]
    new = torch.full((n,), -1, device="cuda")
    new[old] = torch.arange(old.numel(), device="cuda")
    sizes = torch.bincount(gid[old], minlength=len(specs)).tolist()
    u, v = new[u], new[v]
    keep = (u >= 0) & (v >= 0)
    u, v, w = u[keep], v[keep], w[keep]
    n = old.numel()
    if raw:
        more = _ints(g, 0, u.numel(), u.numel() // 8)
        loops = _ints(g, 0, n, n // 16)
        src = torch.cat([u, v, u[more], v[more], loops])
        dst = torch.cat([v, u, v[more], u[more], loops])
        extra = _ints(g, 1, wmax + 1, more.numel())
        w = torch.cat([w, w, extra, extra, _ints(g, 1, wmax + 1, loops.numel())])
        order = torch.argsort(src + _uniform(g, (src.numel(),)))
        src, dst, w = src[order], dst[order], w[order]
    else:
        key, order = torch.sort(torch.cat([u, v]) * n + torch.cat([v, u]))
        src, dst, w = key // n, key % n, torch.cat([w, w])[order]
    row = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    row[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    out, at = [], 0
    lo = row[torch.tensor([0] + sizes, device="cuda").cumsum(0)].tolist()
    for k, s in enumerate(sizes):
        out.append(((row[at:at + s + 1] - lo[k]).to(torch.int32), (dst[lo[k]:lo[k + 1]] - at).to(torch.int32),
                    w[lo[k]:lo[k + 1]].clone()))
        at += s
    return out


def _to_host(dev):
    rp, col, w = (x.cpu().numpy() for x in dev)
    return SimpleNamespace(n=rp.size - 1, row_ptr=rp, col=col, w=w)


def _mixed(case):
    """Specs of a batch or of a set of requests: families in turn, mean
    degrees over 8..32, sizes evenly spread over the logarithm of the range,
    in shuffled order."""
    specs = []
    for k in range(case["count"]):
        x = (k + 0.5) / case["count"]
        d = 8 + 7 * k % 25
        if case["kind"] == "batch":
            n = int(case["nmin"] * (case["nmax"] / case["nmin"]) ** x)
        else:
            n = max(64, int(2 * case["mmin"] * (case["mmax"] / case["mmin"]) ** x / d))
        specs.append((("planted", "er", "chung_lu")[k % 3], n, d, 0))
    random.Random(case["count"]).shuffle(specs)
    return specs


def _inputs(case, seed):
    """The case's graphs as device (row_ptr, col, w) tuples."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if case["kind"] == "solve":
        specs = [(case["family"], case["n"], case["degree"], case["core"])]
        return _graphs(specs, case["wmax"], g, raw=case["raw"])
    return _graphs(_mixed(case), case["wmax"], g)


# ------------------------------------------------------------ the cases' calls
def prepare(case, seed):
    graphs = _inputs(case, seed)
    options = {} if case.get("heuristic", True) else {"heuristic_min_n": 0}
    ctx = mc.Context(0, **options)
    s = SimpleNamespace(kind=case["kind"], ctx=ctx, host=None, dev=None, side=not case.get("core"))
    if case["kind"] == "serve":
        s.host = [_to_host(d) for d in graphs]
        s.server = mc.Server(ctx, hbm_bytes=8 << 30, max_inflight=256, max_request_n=max(h.n for h in s.host),
                             max_request_nnz=max(h.col.size for h in s.host), solo_slots=2)
        return s
    if case["kind"] == "batch":
        s.dev = graphs
        size = ctx.batch_workspace_bytes(devs=graphs)
        if case["host"]:
            s.dev, s.host = None, [_to_host(d) for d in graphs]
            size = ctx.batch_workspace_bytes(graphs=s.host)
    else:
        s.dev = graphs[0]
        size = ctx.workspace_bytes(s.dev[0].numel() - 1, s.dev[1].numel())
        if case["host"]:
            s.dev, s.host = None, _to_host(graphs[0])
    s.workspace = torch.empty(size, dtype=torch.uint8, device="cuda")
    return s


def run(state):
    if state.kind == "solve":
        if state.side:
            return state.ctx.mincut(state.host, dev=state.dev, workspace=state.workspace)
        value, _, stats = state.ctx.mincut(dev=state.dev, workspace=state.workspace, want_side=False,
                                           return_stats=True)
        return value, stats["n_input"], stats["m_input"]
    if state.kind == "batch":
        values, sides = state.ctx.mincut_batch(graphs=state.host, devs=state.dev, workspace=state.workspace)
        return values, np.concatenate(sides)
    tickets = [state.server.submit(h) for h in state.host]
    answers = [None] * len(tickets)
    while any(a is None for a in answers):
        state.server.step()
        for i, t in enumerate(tickets):
            if answers[i] is None:
                answers[i] = state.server.poll(t)
    return np.array([a[0] for a in answers]), np.concatenate([a[1] for a in answers])


def work(case):
    """Every entry (target and weight) and row offset read once, one side
    byte per vertex written; one addition per entry. Sizes before the core is
    taken; of a batch or of requests the mean over the log-uniform range."""
    if case["kind"] == "solve":
        n, entries = case["n"], case["n"] * case["degree"]
    elif case["kind"] == "batch":
        lo, hi = case["nmin"], case["nmax"]
        n = case["count"] * (hi - lo) / math.log(hi / lo)
        entries = 20 * n
    else:
        lo, hi = case["mmin"], case["mmax"]
        entries = 2 * case["count"] * (hi - lo) / math.log(hi / lo)
        n = entries / 18
    return {"bytes": 12.0 * entries + 5.0 * n, "flops": float(entries)}


def exact(case, seed):
    """The minimum cut's value by repeated maximum-adjacency orderings with
    contraction (Nagamochi, Ono and Ibaraki) in int64 numpy, for small
    inputs; a side has no value of its own (any minimum cut's will do)."""
    size = case["n"] if case["kind"] == "solve" else sum(s[1] for s in _mixed(case))
    if size > 20000 or case.get("core"):
        return None
    values = [_min_cut(_to_host(d)) for d in _inputs(case, seed)]
    return (values[0], None) if case["kind"] == "solve" else (np.array(values, np.int64), None)


def _min_cut(h):
    n, rp, w = h.n, h.row_ptr.astype(np.int64), h.w
    src, dst = np.repeat(np.arange(n), np.diff(rp)), h.col.astype(np.int64)
    lam = None
    while True:
        # simple graph in row order: loops dropped, parallel entries summed
        keep = src != dst
        key, at = np.unique(src[keep] * n + dst[keep], return_inverse=True)
        total = np.zeros(key.size, np.int64)
        np.add.at(total, at, w[keep])
        src, dst, w = key // n, key % n, total
        rp = np.searchsorted(src, np.arange(n + 1))
        deg = np.zeros(n, np.int64)
        np.add.at(deg, src, w)
        lam = int(deg.min()) if lam is None else min(lam, int(deg.min()))
        if n == 2:
            return lam
        # one ordering: r of unvisited vertices, pairs that lam certifies
        r, alpha, parent = np.zeros(n, np.int64), 0, np.arange(n)

        def find(x):
            while parent[x] != x:
                parent[x] = parent[parent[x]]
                x = parent[x]
            return x
        for i in range(n):
            x = int(np.argmax(r))
            alpha += int(deg[x]) - 2 * int(r[x])
            r[x] = -1
            if i < n - 1:
                lam = min(lam, alpha)
            y = dst[rp[x]:rp[x + 1]]
            open_ = r[y] >= 0
            y, wy = y[open_], w[rp[x]:rp[x + 1]][open_]
            r[y] += wy
            for z in y[r[y] >= lam]:
                a, b = find(x), find(int(z))
                if a != b:
                    parent[max(a, b)] = min(a, b)
        label = np.array([find(x) for x in range(n)])
        roots, label = np.unique(label, return_inverse=True)
        if roots.size == 1:
            return lam
        n, src, dst = roots.size, label[src], label[dst]
