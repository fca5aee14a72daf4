"""Calls that fail under a pool cap while their search for shortest paths runs
beside the extension, each followed at once by a call on another graph that
fits the same buffers."""
import numpy as np
import pytest

from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import check_tp, say

pytestmark = pytest.mark.gpu


def _guards(n, step):
    """n vertices in a row; every step-th one may leave to the exit."""
    edges = [(i, i + 1) for i in range(n - 1)] + [(i, n - 1) for i in range(0, n - 2, step)]
    return cfggen.from_edges(n, edges, name=f"guards_{n}_{step}")


@pytest.mark.parametrize("n", [60, 300])
def test_next_call_after_a_refused_one(n):
    w = tpg.Workspace()
    tpg.test_paths(tpg.load_cfg(_guards(n, 1)), ws=w)
    full = w.bytes
    w.close()
    for part in (0.2, 0.4, 0.6, 0.8):
        w = tpg.Workspace()
        check_tp(_guards(n // 2, 2), w=w)  # room for the smaller graphs
        for step in (2, 3, 5):
            say("case", n, part, step)
            try:
                tpg.test_paths(tpg.load_cfg(_guards(n, 1)), ws=w, pool_cap=max(w.bytes, int(part * full)))
            except tpg.TpgError as e:
                assert e.name == "TPG_ERR_CAPACITY"
            check_tp(_guards(n // 2, step), w=w)
        w.close()


def test_batch_after_a_refused_one():
    gs = [_guards(40 + k, 1 + k % 3) for k in range(12)]
    hs = [tpg.load_cfg(g) for g in gs]
    ref, _ = tpg.batch_test_paths(hs)
    big = [tpg.load_cfg(_guards(300, 1))] + hs
    w = tpg.Workspace()
    for _ in range(4):  # direct, recorded, captured, replayed
        with pytest.raises(tpg.TpgError):
            tpg.batch_test_paths(big, ws=w, pool_cap=max(w.bytes, 1 << 20))
        got, _ = tpg.batch_test_paths(hs, ws=w)
        for a, b in ((got.pp, ref.pp), (got.tp, ref.tp)):
            assert np.array_equal(a.offsets, b.offsets) and np.array_equal(a.vertices, b.vertices)
    w.close()
