"""Unions past the one-workgroup forms of the batched call: more than 16384
vertices or arcs (roots and arcs placed around a scan), 1024 or more chains that
start cycles (256 threads each), in caller order, against single calls."""
import numpy as np
import pytest

from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _line(k):
    return cfggen.from_edges(k, [(i, i + 1) for i in range(k - 1)], name=f"line_{k}")


def _members(count):
    gs = [cfggen.batch_member_cfg(cfggen.C3_SEED_BASE + s) for s in range(40)]
    gs += [cfggen.loop_diamond_chain(k) for k in (1, 2, 6)] + [_line(1), _line(9)]
    return [gs[(7 * i) % len(gs)] for i in range(count)]


# 16384 vertices are lines' last and first; then arcs alone, then all of it
@pytest.mark.parametrize("graphs", ["lines_16383", "lines_16384", "lines_16385", "mixed_600",
                                    "mixed_2000"])
def test_batch_equals_single_calls(graphs):
    say("case large union", graphs)
    n = int(graphs.split("_")[1])
    gs = [_line(63)] * (n // 63) + ([_line(n % 63)] if n % 63 else []) \
        if graphs.startswith("lines") else _members(n)
    hs = {}
    for g in gs:
        if id(g) not in hs:
            hs[id(g)] = tpg.load_cfg(g)
    w, one = tpg.Workspace(), tpg.Workspace()
    want = {}
    for k, h in hs.items():
        want[k] = tpg.test_paths(h, ws=one)[:2]
    loaded = [tpg.load_cfg(g) for g in gs]
    for turn in range(3):
        r, _ = tpg.batch_test_paths(loaded, ws=w)
        for i, g in enumerate(gs):
            for (off, vtx), ref in zip(r.graph(i), want[id(g)]):
                assert np.array_equal(off, ref.offsets) and np.array_equal(vtx, ref.vertices), (
                    turn, i, g.name)
    w.close()
    one.close()
