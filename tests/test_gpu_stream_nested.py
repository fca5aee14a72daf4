"""A streamed chunk's arrays while its callback makes other calls on the same
workspace: streamed, single and batched, larger and smaller ones, under a cap."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import same, say

pytestmark = pytest.mark.gpu


def _arrays(c):
    off = np.ctypeslib.as_array(ctypes.cast(c.offsets, ctypes.POINTER(ctypes.c_int64)),
                                shape=(c.n_paths + 1,))
    vtx = np.ctypeslib.as_array(ctypes.cast(c.vertices, ctypes.POINTER(ctypes.c_int32)),
                                shape=(max(c.n_vertices, 1),))[:c.n_vertices]
    return off, vtx


@pytest.mark.parametrize("inner", ["stream", "large stream", "single", "batch", "capped"])
@pytest.mark.parametrize("outer", [6, 9])
def test_chunk_outlives_calls_of_its_callback(outer, inner):
    say("case", outer, inner)
    w = tpg.Workspace()
    g = tpg.load_cfg(cfggen.loop_diamond_chain(outer))
    h = tpg.load_cfg(cfggen.loop_diamond_chain(9 if inner == "large stream" else 5))
    want_h, _ = tpg.prime_paths(h)
    got = []

    def other():
        if inner == "batch":
            r, _ = tpg.batch_test_paths([h, h, g], ws=w)
            off, vtx = r.graph(1)[0]
            return np.array_equal(off, want_h.offsets) and np.array_equal(vtx, want_h.vertices)
        if "stream" in inner:
            parts = []
            tpg.prime_paths_stream(h, lambda c, a, b: parts.append(c.vertices), ws=w, chunk_vertices=8)
            return np.array_equal(np.concatenate(parts), want_h.vertices)
        if inner == "capped":
            with pytest.raises(tpg.TpgError):
                tpg.prime_paths(h, ws=w, pool_cap=1000)
        return same(tpg.prime_paths(h, ws=w)[0], want_h)

    def on_chunk(_ctx, p, first, end):
        off, vtx = _arrays(p.contents)
        before = off.copy(), vtx.copy()
        ok = other()
        off, vtx = _arrays(p.contents)
        ok = ok and np.array_equal(off, before[0]) and np.array_equal(vtx, before[1])
        got.append(vtx.copy())
        return 0 if ok else 1

    want = oracle.prime_paths_local(cfggen.loop_diamond_chain(outer), 0, 3 * outer + 5)[0]
    for _ in range(2):
        got.clear()
        o = tpg._opts(w, tpg.TPG_STREAM, None, None)
        o.chunk_vertices = 10
        cb = tpg._CHUNK_FN(on_chunk)
        o.on_chunk = cb
        out = tpg._Paths()
        tpg._check(tpg.lib().tpg_prime_paths(g.handle, ctypes.byref(o), ctypes.byref(out)))
        assert np.array_equal(np.concatenate(got), want.vertices) and out.n_paths == len(want)
    w.close()
