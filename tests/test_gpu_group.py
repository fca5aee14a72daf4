"""Prime paths grouped by last vertex (TPG_ORDER_BY_LAST): sets around a wave's
64 paths and a tile's 1024, one key for all of them or as many keys as a graph
can have, against a stable sort of the canonical set."""
import numpy as np
import pytest

from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import say, ws
from tests.test_gpu_narrow import _fans

pytestmark = pytest.mark.gpu


def _check(g, load_flags=0):
    say("case group", g.name)
    h = tpg.load_cfg(g, load_flags)
    plain, _ = tpg.prime_paths(h, ws=ws())
    got, _ = tpg.prime_paths(h, ws=ws(), flags=tpg.TPG_ORDER_BY_LAST)
    rows = plain.tolist()
    assert got.tolist() == sorted(rows, key=lambda r: r[-1])  # stable
    return len(rows)


# one end for all paths
@pytest.mark.parametrize("widths", [(2,), (21, 3), (32, 2), (13, 5), (31, 33), (32, 32),
                                    (25, 41), (32, 32, 3)])
def test_one_key(widths):
    assert _check(_fans(widths)[0]) == int(np.prod(widths))


# every vertex ends paths: cycles of the loop start everywhere
@pytest.mark.parametrize("widths", [(2,), (5, 3), (9, 10), (12, 12, 2)])
def test_loops(widths):
    _check(_fans(widths, back=True)[0])


# a ring, up to the
# largest size: n paths and n keys
@pytest.mark.parametrize("n", [2, 3, 64, 65, 1024, 1025, 4096])
def test_rings(n):
    g = cfggen.from_edges(n, [(v, (v + 1) % n) for v in range(n)], name=f"ring_{n}")
    assert _check(g, tpg.TPG_LOAD_ANY_DIGRAPH) == n
