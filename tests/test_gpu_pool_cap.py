"""Pool caps that hold what a call needs and little more: shallow graphs of many
vertices, whose prefix and suffix rows are short."""
import pytest

import oracle
from paper_2210_16998_amd import tpg
from tests.gpu_util import check_tp, same, say
from tests.test_gpu_deep import _guards, _switches

pytestmark = pytest.mark.gpu


# 72 and 5 MB; the rows have 20 k and 5 k entries
@pytest.mark.parametrize("a,b,mb", [(64, 62, 80), (30, 30, 6)])
def test_rows_of_shallow_graphs_fit_the_cap(a, b, mb):
    g = _switches(a, b)
    say("case", g.name)
    w = tpg.Workspace()
    pp, tp, _ = tpg.test_paths(tpg.load_cfg(g), ws=w, pool_cap=mb << 20)
    assert w.bytes <= mb << 20
    ref = oracle.prime_paths_local(g, 0, g.n)[0]
    assert same(pp, ref) and same(tp, oracle.test_paths(g, ref)[0])
    w.close()


def test_rows_of_a_batch_fit_the_cap():
    gs = [_switches(30, 30) for _ in range(8)] + [_guards(100) for _ in range(8)]
    w = tpg.Workspace()
    r, _ = tpg.batch_test_paths([tpg.load_cfg(g) for g in gs], ws=w, pool_cap=48 << 20)
    for k in (0, 7, 8, 15):
        pp = oracle.prime_paths_local(gs[k], 0, gs[k].n)[0]
        for (off, vtx), want in zip(r.graph(k), (pp, oracle.test_paths(gs[k], pp)[0])):
            assert (off == want.offsets).all() and (vtx == want.vertices).all()
    w.close()


@pytest.mark.parametrize("n", [1, 2, 64, 65, 300])
def test_rows_next_to_each_other(n):
    """Rows of every length from one vertex to all of them."""
    say("case", n)
    check_tp(_guards(n + 2))
    check_tp(_guards(n + 2, True))
