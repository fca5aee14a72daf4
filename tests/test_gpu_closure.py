"""Strongly connected components of single graphs around the sizes of the
closure over chains (64, 128, 256 and 512 chains; beyond it the search), with
ids out of order along the lines, against the oracle."""
import numpy as np
import pytest

from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import say
from tests.test_gpu_scc import _check_scc

pytestmark = pytest.mark.gpu


def _digraph(seed, n, arcs):
    rng = np.random.default_rng(seed)
    e = {(int(a), int(b)) for a, b in rng.integers(0, n, (arcs, 2))}
    return cfggen.from_edges(n, sorted(e), name=f"digraph_{seed}_{n}_{arcs}")


def _check(g):
    say("case closure", g.name)
    _check_scc(g, tpg.TPG_LOAD_ANY_DIGRAPH)


# two arcs a vertex: few lines, so about n chains; one giant component or many
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 256, 258, 511, 513, 520, 600])
def test_digraphs(n):
    for seed, per in ((1, 0.8), (2, 1.2), (3, 2.5)):
        _check(_digraph(seed * 1000 + n, n, int(per * n) + 1))


# long lines, numbered at random: rings on lines, lines between rings
@pytest.mark.parametrize("n", [10, 300, 4096])
def test_lines_and_rings(n):
    rng = np.random.default_rng(n)
    perm = rng.permutation(n)
    cuts = np.sort(rng.choice(np.arange(1, n), min(6, n - 1), replace=False))
    edges = [(int(perm[i]), int(perm[i + 1])) for i in range(n - 1)]
    for a, b in zip(cuts[:-1:2], cuts[1::2]):
        edges.append((int(perm[b]), int(perm[a])))
    _check(cfggen.from_edges(n, sorted(set(edges)), name=f"lines_{n}"))
    _check(cfggen.from_edges(n, [(int(perm[i]), int(perm[(i + 1) % n])) for i in range(n)],
                             name=f"ring_{n}"))
