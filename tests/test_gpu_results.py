"""Host results of one workspace that are kept while later calls run: small
ones, which pass through pinned memory together, ones that outgrow it (4 MiB)
and its first sizes, a refused call in between, and rows written before the
host knows their number (up to 4 Mi entries) next to larger sets."""
import numpy as np
import pytest

import oracle
from paper_2210_16998_amd import tpg
from tests.gpu_util import say
from tests.test_gpu_narrow import _fans

pytestmark = pytest.mark.gpu


def _want(widths, back):
    g, _ = _fans(widths, back)
    pp = oracle.prime_paths(g)[0]
    return g, pp, oracle.test_paths(g, pp)[0]


def _same(got, want):
    return (np.array_equal(got.offsets, np.asarray(want.offsets))
            and np.array_equal(got.vertices, np.asarray(want.vertices)))


# 6 to 15 entries a path: 2 KB, 0.3 MB, 5 MB, 0.3 MB, 26 MB and 2 KB of rows
SIZES = [((2, 3), False), ((9, 10, 9), True), ((32, 32, 32), False), ((12, 12, 2), True),
         ((28, 28, 28), True), ((2, 3), True)]


@pytest.mark.parametrize("order", [(0, 1, 2, 3, 4, 5), (4, 0, 2, 5, 1, 3), (5, 4, 3, 2, 1, 0)])
def test_kept_results_of_many_calls(order):
    w = tpg.Workspace()
    kept = []
    for i in order:
        g, pp, tp = _want(*SIZES[i])
        say("case", g.name, SIZES[i][1])
        h = tpg.load_cfg(g)
        kept.append((tpg.test_paths(h, ws=w)[:2], (pp, tp)))
        kept.append((tpg.prime_paths(h, ws=w)[:1], (pp,)))
        with pytest.raises(Exception):
            tpg.test_paths(h, ws=w, pool_cap=1)
        chunks = []
        tpg.prime_paths_stream(h, lambda c, a, b: chunks.append(c), ws=w, chunk_vertices=8)
        assert np.array_equal(np.concatenate([c.vertices for c in chunks]), np.asarray(pp.vertices))
    w.close()
    for got, want in kept:
        assert all(_same(a, b) for a, b in zip(got, want))
    view = kept[0][0][0].vertices
    text = view.tolist()
    kept.clear()
    assert view.tolist() == text  # outlives the result it belongs to


@pytest.mark.parametrize("flags", [0, tpg.TPG_OUT_DEVICE])
def test_batches_around_the_room_ahead(flags):
    """One union of small graphs, then one with a large member."""
    w = tpg.Workspace()
    for which in ([0, 1], [0, 3, 5], [0, 4, 5], [1, 0]):
        sets = [_want(*SIZES[i]) for i in which]
        hs = [tpg.load_cfg(g) for g, _, _ in sets]
        for _ in range(4):  # direct, recorded, captured, replayed
            r, _st = tpg.batch_test_paths(hs, ws=w, flags=flags)
            if flags:
                continue
            for k, (_, pp, tp) in enumerate(sets):
                for (off, vtx), ref in zip(r.graph(k), (pp, tp)):
                    assert np.array_equal(off, np.asarray(ref.offsets)), which
                    assert np.array_equal(vtx, np.asarray(ref.vertices)), which
        if flags:
            n = [(len(pp), len(tp)) for _, pp, tp in sets]
            assert np.array_equal(np.diff(r.pp_first), [a for a, _ in n])
            assert np.array_equal(np.diff(r.tp_first), [b for _, b in n])
