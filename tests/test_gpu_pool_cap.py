"""Pool caps that hold what a call needs and little more: shallow graphs of many
vertices, whose prefix and suffix rows are short, and calls that only fit with
no buffer larger than it has to be."""
import ctypes

import pytest

import oracle
from paper_2210_16998_amd import cfggen, tpg
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


def _graph(name):
    if name.startswith("guards"):
        return _guards(int(name[6:]))
    return cfggen.c1_cfg() if name == "c1" else cfggen.loop_diamond_chain(int(name[4:]))


def _call(kind, h, w, cap):
    if kind == "tp":
        return tpg.test_paths(h, ws=w, pool_cap=cap)[:2]
    if kind == "cover":
        return tpg.test_paths(h, ws=w, pool_cap=cap, flags=tpg.TPG_TP_GREEDY)[:2]
    if kind == "last":
        return tpg.prime_paths(h, ws=w, pool_cap=cap, flags=tpg.TPG_ORDER_BY_LAST)[:1]
    if kind == "stream":
        chunks = []
        tpg.prime_paths_stream(h, lambda c, a, b: chunks.append(c), ws=w, pool_cap=cap)
        return chunks
    return tpg.prime_paths(h, ws=w, pool_cap=cap)[:1]


# KB that a call fits in if nothing is to spare; what it takes with room ahead,
# guesses and growth by a quarter is more (in brackets)
@pytest.mark.parametrize("name,kind,kb", [
    ("guards100", "pp", 355), ("guards100", "tp", 432), ("guards100", "cover", 469), ("guards100", "last", 382), ("guards100", "stream", 336),  # (399 569 562 424 381)
    ("guards300", "pp", 2630), ("guards300", "tp", 3170), ("guards300", "cover", 3370), ("guards300", "stream", 1107),  # (2903 4382 4202 1193)
    ("loop10", "pp", 7377), ("loop10", "last", 11400), ("loop10", "tp", 12000), ("loop10", "cover", 15000),  # (7660 11585 12937 15213)
    ("c1", "pp", 166), ("c1", "tp", 183), ("c1", "cover", 202)])  # (191 204 215)
def test_cap_with_nothing_to_spare(name, kind, kb):
    g, cap = _graph(name), kb * 1000
    say("case", name, kind)
    h, w = tpg.load_cfg(g), tpg.Workspace()
    want = _call(kind, h, None, 0)
    for _ in range(3):  # refused with room to spare and run again; without from the start
        got = _call(kind, h, w, cap)
        assert w.bytes <= cap
        assert len(got) == len(want) and all(same(a, b) for a, b in zip(got, want))
    if kind in ("pp", "tp"):
        pp = oracle.prime_paths_local(g, 0, g.n)[0]
        assert same(got[0], pp) and (kind == "pp" or same(got[1], oracle.test_paths(g, pp)[0]))
    with pytest.raises(tpg.TpgError) as e:
        _call(kind, h, w, max(1000, w.bytes // 2))
    assert e.value.name == "TPG_ERR_CAPACITY"
    got = _call(kind, h, w, 0)
    assert all(same(a, b) for a, b in zip(got, want))
    w.close()


def test_batch_with_nothing_to_spare():
    """What holds such a batch with room to spare is 17.4 MB."""
    gs = [cfggen.batch_member_cfg(cfggen.C3_SEED_BASE + s) for s in range(60)] + [_guards(200)]
    hs, w, cap = [tpg.load_cfg(g) for g in gs], tpg.Workspace(), 12 << 20
    ref, _ = tpg.batch_test_paths(hs)
    for _ in range(4):
        r, _ = tpg.batch_test_paths(hs, ws=w, pool_cap=cap)
        assert w.bytes <= cap and same(r.pp, ref.pp) and same(r.tp, ref.tp)
        assert (r.pp_first == ref.pp_first).all() and (r.tp_first == ref.tp_first).all()
    w.close()


# KB as above
@pytest.mark.parametrize("fn,n,kb", [("merged_pps", 3, 2000), ("scc_paths", 3, 900),
                                     ("scc_internal_pps", 1, 2000)])  # (6236 973 2137)
def test_components_with_nothing_to_spare(fn, n, kb):
    g, w = tpg.load_cfg(cfggen.loop_diamond_chain(8)), tpg.Workspace()
    want = getattr(tpg, fn)(g)
    for _ in range(2):
        outs = [tpg._Paths() for _ in range(n)]
        o = tpg._opts(w, 0, None, None, kb * 1000)
        tpg._check(getattr(tpg.lib(), "tpg_" + fn)(g.handle, ctypes.byref(o), *map(ctypes.byref, outs)))
        assert w.bytes <= kb * 1000
        assert all(same(tpg._wrap(a), b) for a, b in zip(outs, want if n > 1 else [want]))
    w.close()
