"""Prime-path rows around the 32 depths that a wave writes at once, paths of
very different lengths side by side in a wave, in the writer's staged form (up
to 2048 vertices) and past it."""
import numpy as np
import pytest

import oracle
from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import say, ws

pytestmark = pytest.mark.gpu


def _comb(lengths):
    """Lines of the given lengths side by side between entry and exit."""
    edges, n = [], 1
    for k in lengths:
        stops = [0] + list(range(n, n + k))
        n += k
        edges += list(zip(stops[:-1], stops[1:]))
    ends = np.cumsum(lengths)
    edges += [(int(e), n) for e in ends]
    return cfggen.from_edges(n + 1, edges, name=f"comb_{len(lengths)}_{n + 1}")


@pytest.mark.parametrize("lengths", [(30,), (29, 30, 31, 61, 62, 63), tuple(range(1, 60)),
                                     (1, 2044), (1, 1, 2045), (700, 3, 900, 441), (4000, 5)])
def test_rows(lengths):
    g = _comb(lengths)
    say("case rows", g.name)
    pp, tp, _ = tpg.test_paths(tpg.load_cfg(g), ws=ws())
    rp = oracle.prime_paths(g)[0]
    for p in (pp, tp):  # every path runs from the entry to the exit
        assert np.array_equal(p.offsets, np.asarray(rp.offsets))
        assert np.array_equal(p.vertices, np.asarray(rp.vertices))
