"""GPU tests of the order in which a round tries its tests, read from the lines
that MC_DEBUG prints (in a process of its own, whose stderr is caught)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# 33 x 34 cliques of 60 on a torus, five unit edges between neighbours: the
# smallest degree is 59, the smallest cut 20, around one clique. The heuristic
# finds it; its coarse graph, the torus, resists the tests.
CLIQUES = """
import numpy as np
import gen
import oracle
import paper_2609_07204_amd as mc
a, b, s = 33, 34, 60
r = np.random.default_rng(4)
i, j = np.triu_indices(s, 1)
k = np.arange(a * b).reshape(a, b)
us, vs = [(k.reshape(-1, 1) * s + i).ravel()], [(k.reshape(-1, 1) * s + j).ravel()]
for axis in (0, 1):
    for e in range(5):
        us.append(k.ravel() * s + 10 * axis + e)
        vs.append(np.roll(k, 1, axis).ravel() * s + 20 + 10 * axis + e)
n = a * b * s
p = r.permutation(n)
u, v = p[np.concatenate(us)], p[np.concatenate(vs)]
g = gen.from_edges(n, u, v, np.ones(u.size, np.int64))
lam, side = mc.Context(0).mincut(g)
assert lam == 20 and oracle.cut_value(g, side) == 20, lam
"""


def debug_lines(code):
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True,
                       timeout=100, env=dict(os.environ, MC_DEBUG="1", PYTHONPATH=ROOT))
    assert p.returncode == 0, p.stderr[-2000:]
    return [l for l in p.stderr.splitlines() if l.startswith("[mc]")]


def test_subgraphs_are_tried_again_at_the_heuristics_bound():
    lines = debug_lines(CLIQUES)
    n = 33 * 34 * 60
    print("\n".join(lines))
    tried = [k for k, l in enumerate(lines) if "edge-disjoint subgraphs: n=%d " % n in l]
    # at the smallest degree, then at the heuristic's bound, before a lower one is looked for
    assert len(tried) >= 2 and "lam=59" in lines[tried[0]] and "lam=20" in lines[tried[1]], lines
    assert not any("threshold" in l for l in lines[:tried[1]]), lines


# passes with their state in LDS report their own steps, not those of an earlier launch
PRIVATE = """
import numpy as np
import gen
import paper_2609_07204_amd as mc
r = np.random.default_rng(1)
for n in (20000, 1500, 1500):
    p = r.permutation(n)
    u, v = np.concatenate([p, r.integers(0, n, 2 * n)]), np.concatenate([np.roll(p, 1), r.integers(0, n, 2 * n)])
    g = gen.from_edges(n, u, v, r.integers(50, 100, u.size))
    mc.Context(0, capforest_mode=0, capforest_passes=2, heuristic_min_n=0, pr_tri_deg_cap=0).mincut(g)
"""


def test_lds_passes_report_their_steps():
    import re
    lines = [l for l in debug_lines(PRIVATE) if "passes=2" in l]
    seen = 0
    for l in lines:
        n, steps, singles, scans, batch = (int(re.search(p, l).group(1)) for p in (
            r" n=(\d+) ", r"steps max (\d+) ", r"singles max (\d+) ", r"scans max (\d+) ", r"maxbatch (\d+)"))
        assert 1 <= scans <= n and 1 <= batch <= scans and 1 <= singles <= steps <= scans, l
        seen += n <= 16256
    assert seen, lines
