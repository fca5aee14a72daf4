"""Longest-first covering on graphs stretched to given sizes: rows whose windows
cross the 64 positions that a wave takes at once, and sizes around the line
(n = 426) between four paths and one path per workgroup, up to the largest
graph; loops around diamonds, whose paths cover each other."""
import numpy as np
import pytest

import oracle
from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import same, say

pytestmark = pytest.mark.gpu


def _stretched(seed, n):
    """A small random CFG with vertices put on its arcs until it has n."""
    rng = np.random.default_rng(seed)
    base = cfggen.random_small_cfg(60_000 + seed, 7, extra=5)
    edges = base.edges()
    add = rng.multinomial(n - base.n, np.ones(len(edges)) / len(edges))
    out, k = [], base.n
    for (a, b), m in zip(edges, add):
        stops = [a] + list(range(k, k + int(m))) + [b]
        k += int(m)
        out += list(zip(stops[:-1], stops[1:]))
    return cfggen.from_edges(n, out, base.entry, base.exit, name=f"stretched_{seed}_{n}")


def _check(g, w):
    say("case cover", g.name)
    pp, tp, st = tpg.test_paths(tpg.load_cfg(g), ws=w, flags=tpg.TPG_TP_GREEDY)
    rp = oracle.prime_paths(g)[0]
    rt = oracle.test_paths_greedy(g, rp)
    assert same(pp, rp) and same(tp, rt), g.name
    assert st["n_tp"] == len(rt)


@pytest.mark.parametrize("n", [20, 63, 64, 65, 127, 129, 200, 425, 426, 427, 428, 1000, 4096])
def test_sizes(n):
    w = tpg.Workspace()
    for seed in range(6) if n <= 1000 else (1, 3):
        _check(_stretched(seed, n), w)
    w.close()


@pytest.mark.parametrize("k", [1, 2, 3, 5, 7])
def test_loops_in_a_new_workspace(k):
    w = tpg.Workspace()
    _check(cfggen.loop_diamond_chain(k), w)
    w.close()
