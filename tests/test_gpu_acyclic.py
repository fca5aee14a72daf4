"""Graphs without a cycle, whose test paths are their prime paths: sizes around
the 16 bytes that a lane copies and around the rows written ahead, one cycle
more or less, alone, covered, streamed, in batches of acyclic and mixed unions,
and under a cap with nothing to spare."""
import random

import numpy as np
import pytest

import oracle
from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import check_tp, same, say, ws
from tests.test_gpu_deep import _guards, _switches
from tests.test_gpu_narrow import _fans

pytestmark = pytest.mark.gpu


def _dag(seed, n, extra, loop=False):
    """Random arcs to later vertices, every vertex on a way through; loop: one arc
    back."""
    r = random.Random(seed)
    e = {(r.randrange(v), v) for v in range(1, n)} | {(v, r.randrange(v + 1, n)) for v in range(n - 1)}
    while extra > 0:
        a, b = sorted(r.sample(range(n), 2))
        e.add((a, b))
        extra -= 1
    if loop and n > 3:
        a, b = sorted(r.sample(range(1, n - 1), 2))
        e.add((b, a))
    return cfggen.from_edges(n, sorted(e), name=f"dag_{seed}_{n}_{loop}")


@pytest.mark.parametrize("loop", [False, True])
@pytest.mark.parametrize("n", [2, 3, 4, 5, 6, 7, 9, 12, 18, 25, 33, 60])
def test_random_graphs(n, loop):
    for seed in range(6):
        g = _dag(seed, n, n // 3, loop)
        say("case", g.name)
        check_tp(g)
        check_tp(g, tpg.TPG_FORCE_TWO_PASS)


@pytest.mark.parametrize("g", [cfggen.from_edges(1, [], 0, 0), _guards(40), _switches(9, 7), _dag(1, 40, 30),
                               _dag(2, 30, 12, True), _fans((32, 32, 33))[0]], ids=lambda g: g.name)
def test_options(g):
    say("case", g.name)
    h, pp = tpg.load_cfg(g), oracle.prime_paths_local(g, 0, g.n)[0]
    tp = oracle.test_paths(g, pp)[0]
    for _ in range(2):
        a, b, st = tpg.test_paths(h, ws=ws(), flags=tpg.TPG_DIGEST)
        assert same(a, pp) and same(b, tp) and st["n_tp"] == len(tp) and st["n_tp_vertices"] == len(tp.vertices)
        parts = []
        _, total, _ = tpg.test_paths_stream(h, lambda c, x, y: parts.append(c.vertices), ws=ws(), chunk_paths=7)
        assert np.array_equal(np.concatenate(parts), tp.vertices) and total.digest == b.digest
        a, b, _ = tpg.test_paths(h, ws=ws(), flags=tpg.TPG_TP_GREEDY)
        assert same(a, pp) and same(b, oracle.test_paths_greedy(g, pp))
        a, b, _ = tpg.test_paths(h, ws=ws(), flags=tpg.TPG_OUT_DEVICE)
        assert [a.n_paths, a.n_vertices, b.n_paths, b.n_vertices] == [len(pp), len(pp.vertices), len(tp), len(tp.vertices)]
        views = [v.cpu().numpy() for x in (a, b) for v in x.torch_views()]
        for got, want in zip(views, (pp.offsets, pp.vertices, tp.offsets, tp.vertices)):
            assert np.array_equal(got, want)


@pytest.mark.parametrize("mixed", [False, True])
def test_batches(mixed):
    gs = [_dag(s, 3 + 2 * s, s, mixed and s % 5 == 0) for s in range(30)] + [_guards(90), _switches(10, 9)]
    hs, w = [tpg.load_cfg(g) for g in gs], tpg.Workspace()
    want = [oracle.prime_paths_local(g, 0, g.n)[0] for g in gs]
    want = [(pp, oracle.test_paths(g, pp)[0]) for g, pp in zip(gs, want)]
    for cap in (0, 0, 0, 0, 8 << 20):  # direct, recorded, captured, replayed
        r, st = tpg.batch_test_paths(hs, ws=w, pool_cap=cap)
        for k in range(len(gs)):
            for (off, vtx), ref in zip(r.graph(k), want[k]):
                assert np.array_equal(off, ref.offsets) and np.array_equal(vtx, ref.vertices), (k, cap)
        assert st["n_tp"] == sum(len(t) for _, t in want)
    w.close()


def test_caps_between_the_room_ahead_and_none():
    """4000 paths of 11 entries, 176 KB a set, and 688 KB with room ahead."""
    g = _fans((10, 10, 10, 4))[0]
    h, pp = tpg.load_cfg(g), oracle.prime_paths_local(g, 0, g.n)[0]
    w = tpg.Workspace()
    tpg.test_paths(h, ws=w)
    full = w.bytes
    w.close()
    fits = 0
    for cap in range(full // 2, full + 65536, max(4096, full // 60)):
        w = tpg.Workspace()
        try:
            a, b, _ = tpg.test_paths(h, ws=w, pool_cap=cap)
            assert same(a, pp) and same(b, pp) and w.bytes <= cap
            fits += 1
        except tpg.TpgError as e:
            assert e.name == "TPG_ERR_CAPACITY" and fits == 0
        w.close()
    assert fits > 20
