"""Level and row counts around the one-workgroup forms: levels of the path tree
on both sides of 2048 nodes (swept by one workgroup, or by a launch for two
levels) in one call, more narrow levels than one launch takes (64), and scans
of lengths around 8192 (one step) and 16384 (the last length that one
workgroup takes)."""
import itertools

import numpy as np
import pytest

from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import check_tp, say, ws

pytestmark = pytest.mark.gpu


def _fans(widths, back=False):
    """hub -> widths[0] vertices -> hub -> ...; every path through is prime.
    back: a loop around all of it."""
    edges, hub, n, cols = [(0, 1)], 1, 2, []
    for w in widths:
        mids = list(range(n, n + w))
        n += w + 1
        edges += [(hub, m) for m in mids] + [(m, n - 1) for m in mids]
        cols.append(mids)
        cols.append([n - 1])
        hub = n - 1
    edges.append((hub, n))
    if back:
        edges.append((hub, 1))
    g = cfggen.from_edges(n + 1, edges, name="fans_" + "_".join(map(str, widths)))
    return g, [[0], [1]] + cols + [[n]]


# prime paths, all of equal length: 8192 +- 256, 32768 and its neighbours; level
# sizes from 2 to the same
@pytest.mark.parametrize("widths", [(2,), (32, 32, 2), (31, 33, 2), (33, 32, 2), (32, 8, 31), (33, 31, 16),
                                    (32, 16, 32), (31, 32, 17),
                                    (8, 32, 32), (32, 32, 8), (31, 32, 33), (32, 32, 32),
                                    (32, 32, 33), (2, 2, 2, 32, 32, 4)])
def test_all_paths_of_fans(widths):
    g, cols = _fans(widths)
    say("case", g.name)
    want = np.array(list(itertools.product(*cols)), np.int32)
    n, k = want.shape
    for flags in (0, tpg.TPG_FORCE_TWO_PASS):
        pp, tp, st = tpg.test_paths(tpg.load_cfg(g), ws=ws(), flags=flags)
        for p in (pp, tp):
            assert np.array_equal(np.asarray(p.offsets), k * np.arange(n + 1)), g.name
            assert np.array_equal(np.asarray(p.vertices).reshape(n, k), want), g.name
        assert st["n_pp"] == st["n_tp"] == n


# a new workspace holds 64 nodes a chain and 16 sets a chain to begin with:
# levels that do not fit on both sides of 2048 nodes, inside a launch that takes
# several levels and between launches
@pytest.mark.parametrize("widths", [(2, 2, 2, 2, 2, 2, 2, 2, 2, 2, 2), (16, 16, 8), (32, 32, 32)])
def test_levels_that_do_not_fit_a_new_workspace(widths):
    g, cols = _fans(widths)
    say("case", g.name)
    w = tpg.Workspace()
    want = np.array(list(itertools.product(*cols)), np.int32)
    pp, tp, st = tpg.test_paths(tpg.load_cfg(g), ws=w)
    assert np.array_equal(np.asarray(pp.vertices).reshape(want.shape), want)
    assert np.array_equal(np.asarray(tp.vertices).reshape(want.shape), want)
    assert st["n_pp"] == st["n_tp"] == len(want)


@pytest.mark.parametrize("widths", [(3, 4), (9, 10, 9), (12, 12, 2)])
def test_loops_around_fans(widths):
    g, _ = _fans(widths, back=True)
    say("case", g.name)
    check_tp(g)


# about k levels
@pytest.mark.parametrize("k", [20, 21, 22, 43, 65])
def test_more_narrow_levels_than_a_span(k):
    """A ladder whose rungs all lead to the exit: levels of a few nodes."""
    n = 2 * k + 1
    edges = [(0, 1)]
    for i in range(k):
        a, b = 1 + 2 * i, 2 + 2 * i
        edges.append((a, b))
        edges.append((b, a + 2 if i + 1 < k else n))
        if i + 1 < k:
            edges.append((a, n))
    g = cfggen.from_edges(n + 1, sorted(set(edges)), name=f"ladder_{k}")
    say("case", g.name)
    check_tp(g)
