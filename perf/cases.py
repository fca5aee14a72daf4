"""The calls that a program makes of this framework, each over the sizes, forms
and options it is used with: prime and test paths of one control-flow graph
(CFG), of many CFGs one after another and in one batched call, streamed and
grouped results, covering test paths, the compositional method, and the size
predictor's training gradients.

Path sets are whole numbers and have no rounding; `exact` gives the size
predictor's outputs in 64 bits.
"""
from __future__ import annotations

import functools
import os

import numpy as np

from paper_2210_16998_amd import cfggen, sizer, tpg

# Seeds of the structured ~200-vertex CFGs (Table 1's shape: 36 to 44
# independent paths, 1e5 to 1e6 prime paths).
CFG200 = (2, 5, 6, 14, 15, 19, 29)
# Pool cap of a single large call, as the framework's own benchmark sets it.
POOL_CAP = 64 << 30


def listed():
    return [
        # one small function (3 diamonds, two nested loops; 20 vertices): the
        # fewest paths a call can have, host results
        {"name": "one_small", "kind": "tests", "family": "c1", "host": True},
        # a code base's functions handled one after another on one workspace,
        # every call a graph that the workspace has not just seen
        {"name": "functions_one_by_one", "kind": "each", "count": 48, "base": 3_000_000},
        # a loop around 12 diamonds in the paper's input form, prime paths
        # grouped by the vertex they end at (its output form)
        {"name": "loop_grouped", "kind": "primes", "family": "loop", "k": 12,
         "binarize": True, "by_last": True},
        # one ~200-vertex function: prime and test paths left on the device
        {"name": "cfg212_tests", "kind": "tests", "family": "cfg200", "cfg": 19, "host": False},
        # a long function (1000 vertices, 16-word visited sets)
        {"name": "long_tests", "kind": "tests", "family": "nest", "per_arm": 3, "c0": 1, "c1": 1,
         "c2": 1, "tail": 4, "pad": 1000, "host": False},
        # the high-NPath layout of the benchmark: 400 vertices, 2.3e7 prime
        # paths, 5.4e9 test path entries
        {"name": "stress_tests", "kind": "tests", "family": "nest", "per_arm": 3, "c0": 1, "c1": 1,
         "c2": 1, "tail": 9, "pad": 400, "host": False},
        # prime paths delivered to the host range by range
        {"name": "cfg198_streamed", "kind": "stream", "family": "cfg200", "cfg": 5},
        # fewest test paths: longest-first covering
        {"name": "cfg182_covering", "kind": "cover", "family": "cfg200", "cfg": 29},
        # components, their graph, extracted and merged paths, path types
        {"name": "cfg218_components", "kind": "compose", "family": "cfg200", "cfg": 15},
        # a large code base in one call, sized by the trained predictor
        {"name": "batch_4096", "kind": "batch", "count": 4096, "base": 3_000_000,
         "learned": True, "host": False},
        # a module's functions in one call, host results
        {"name": "batch_64", "kind": "batch", "count": 64, "base": 3_100_000,
         "learned": False, "host": True},
        # one minibatch of the predictor's training: forward and backward
        {"name": "predictor_gradients", "kind": "grad", "rows": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _graph_of(rng, big):
    """A single-CFG shape; `big`: up to the sizes whose results stay on the
    device.  lead: straight-line statements ahead of it."""
    u = rng.random()
    if u < 0.2:
        return {"family": "member", "cfg": rng.randint(3_000_000, 3_099_999)}
    if u < 0.4:
        return _loop_of(rng, 3, 15 if big else 12)
    if u < 0.6:
        return _cfg200_of(rng)
    long = rng.random() < 0.3
    return {"family": "nest", "per_arm": rng.randint(1, 3), "c0": rng.randint(0, 1),
            "c1": rng.randint(0, 1), "c2": rng.randint(0, 1),
            "tail": rng.randint(1, 4 if long or not big else 8),
            "pad": _log_int(rng, 401, 1000) if long and big else _log_int(rng, 100, 400)}


def _loop_of(rng, lo, hi):
    return {"family": "loop", "k": rng.randint(lo, hi), "lead": rng.randint(0, 24)}


def _cfg200_of(rng):
    return {"family": "cfg200", "cfg": rng.choice(CFG200), "lead": rng.randint(1, 24)}


def draw(rng):
    kind = rng.choice(("tests", "tests", "tests", "primes", "primes", "each", "stream", "cover",
                       "compose", "batch", "batch", "grad"))
    if kind == "tests":
        host = rng.random() < 0.3
        return {"kind": kind, "host": host, **_graph_of(rng, not host)}
    if kind == "primes":
        return {"kind": kind, "binarize": rng.random() < 0.5, "by_last": rng.random() < 0.5,
                **_graph_of(rng, True)}
    if kind == "each":
        return {"kind": kind, "count": _log_int(rng, 8, 32),
                "base": 3_000_000 + 1000 * rng.randint(1, 90)}
    if kind == "stream":
        return {"kind": kind, **_graph_of(rng, False)}
    if kind == "cover":
        return {"kind": kind, **(_cfg200_of(rng) if rng.random() < 0.5 else _loop_of(rng, 3, 11))}
    if kind == "compose":
        return {"kind": kind, **(_cfg200_of(rng) if rng.random() < 0.5 else _loop_of(rng, 3, 8))}
    if kind == "batch":
        count = _log_int(rng, 16, 4096)
        return {"kind": kind, "count": count, "base": 3_000_000 + 1000 * rng.randint(1, 90),
                "learned": rng.random() < 0.5, "host": count <= 512 and rng.random() < 0.5}
    return {"kind": "grad", "rows": _log_int(rng, 48, 4096)}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

@functools.lru_cache(maxsize=16)
def _members(base, count):
    return [(g, _siblings(g)) for g in sizer.generate(list(range(base, base + count)), workers=1)]


def _siblings(g):
    """Pairs of successors of one vertex."""
    rows = [r.tolist() for r in np.split(g.col_idx, g.row_ptr[1:-1]) if len(r) > 1]
    return {(a, b) for r in rows for a in r for b in r}


def _base_graph(case):
    f = case["family"]
    if f == "c1":
        return cfggen.c1_cfg()
    if f == "member":
        return cfggen.batch_member_cfg(case["cfg"])
    if f in ("loop", "cfg200"):
        g = cfggen.loop_diamond_chain(case["k"]) if f == "loop" else cfggen.c2_cfg(case["cfg"])
        lead = case.get("lead", 0)
        return cfggen.from_edges(g.n + lead, [(v, v + 1) for v in range(lead)]
                                 + [(a + lead, b + lead) for a, b in g.edges()])
    return cfggen.c5_cfg(case["per_arm"], (case["c0"], case["c1"], case["c2"]), case["tail"],
                         case["pad"])


def _renumbered(g, siblings, rng):
    """The CFG with its inner vertices renumbered a few places apart, as
    another compiler would number the same blocks: neighbouring ids change
    places unless they are successors of one vertex, whose order decides
    between shortest paths.  Same paths, other ids."""
    order = list(range(g.n))  # the vertex at each place
    for flips in (rng.random((4, g.n)) < 0.5).tolist():
        for i in range(1, g.n - 2):
            a, b = order[i], order[i + 1]
            if flips[i] and (a, b) not in siblings:
                order[i], order[i + 1] = b, a
    perm = np.empty(g.n, np.int64)
    perm[order] = np.arange(g.n)
    src, dst = perm[np.repeat(np.arange(g.n), np.diff(g.row_ptr))], perm[g.col_idx]
    by = np.lexsort((dst, src))
    row_ptr = np.zeros(g.n + 1, np.int64)
    np.cumsum(np.bincount(src, minlength=g.n), out=row_ptr[1:])
    return cfggen.CFG(g.n, row_ptr, dst[by].astype(np.int32), 0, g.n - 1, g.name)


def _predictor_inputs(case, seed):
    """Parameters as training starts from, and one minibatch of features and
    exact log1p path counts."""
    rng = np.random.default_rng(seed)
    base = cfggen.C4_SEED_BASE + int(rng.integers(0, 90_000))
    graphs = [tpg.load_cfg(g) for g, _ in _members(base, case["rows"])]
    ws = tpg.Workspace()
    x, t = tpg.features(graphs), sizer.labels(graphs, ws)
    ws.close()
    p = []
    for a, b in ((tpg.MLP_IN, 128), (128, 128), (128, tpg.MLP_OUT)):
        p += [rng.uniform(-1.0, 1.0, a * b) * np.sqrt(6.0 / a), np.zeros(b)]
    mean, std = x.mean(0), x.std(0) + np.float32(1e-6)
    return x, t, np.concatenate(p).astype(np.float32), mean, std


def prepare(case, seed):
    kind = case["kind"]
    s = {"kind": kind}
    if kind == "grad":
        x, t, p, mean, std = _predictor_inputs(case, seed)
        m = tpg.MLP()
        m.set_params(p)
        m.set_normalizer(mean, std)
        return {**s, "mlp": m, "x": x, "t": t}
    rng = np.random.default_rng(seed)
    s["ws"] = tpg.Workspace()
    if kind in ("each", "batch"):
        s["graphs"] = [tpg.load_cfg(_renumbered(g, sib, rng))
                       for g, sib in _members(case["base"], case["count"])]
        if case.get("learned"):
            s["mlp"] = tpg.MLP.load(sizer.DEFAULT_MODEL)
        s["flags"] = tpg.TPG_NO_TIMING | (0 if case.get("host", True) else tpg.TPG_OUT_DEVICE)
        return s
    g = _base_graph(case)
    g = _renumbered(g, _siblings(g), rng)
    s["graph"] = tpg.load_cfg(g, tpg.TPG_LOAD_BINARIZE if case.get("binarize") else 0)
    s["flags"] = tpg.TPG_NO_TIMING | (0 if case.get("host") or kind == "stream"
                                      else tpg.TPG_OUT_DEVICE)
    if case.get("by_last"):
        s["flags"] |= tpg.TPG_ORDER_BY_LAST
    if kind == "cover":
        s["flags"] |= tpg.TPG_TP_GREEDY
    # at most 16 ranges of first vertices
    s["chunk"] = max(32, -(-g.n // 16))
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def _arrays(p, ws):
    if not isinstance(p, tpg.DevicePaths):
        return p.offsets, p.vertices
    views = p.torch_views()
    for v in views:  # they lie in the workspace's memory: it lives as long as they do
        v.workspace = ws
    return views


def run(s):
    kind = s["kind"]
    if kind == "grad":
        g, loss = s["mlp"].gradients(s["x"], s["t"])
        return {"grad": g, "loss": np.float32(loss)}
    if kind in ("tests", "cover"):
        pp, tp, _ = tpg.test_paths(s["graph"], ws=s["ws"], flags=s["flags"], pool_cap=POOL_CAP)
        return {"pp": _arrays(pp, s["ws"]), "tp": _arrays(tp, s["ws"])}
    if kind == "primes":
        pp, _ = tpg.prime_paths(s["graph"], ws=s["ws"], flags=s["flags"], pool_cap=POOL_CAP)
        return {"pp": _arrays(pp, s["ws"])}
    if kind == "each":
        got = [tpg.test_paths(h, ws=s["ws"], flags=s["flags"])[:2] for h in s["graphs"]]
        return {"pp": _joined([a for a, _ in got]), "tp": _joined([b for _, b in got])}
    if kind == "stream":
        chunks = []
        total, _ = tpg.prime_paths_stream(
            s["graph"], lambda c, first, end: chunks.append(c), ws=s["ws"],
            flags=s["flags"], chunk_vertices=s["chunk"])
        return {"pp": _joined(chunks), "digest": np.array(total.digest, np.uint64).view(np.int64)}
    if kind == "compose":
        # results on the device are valid until the workspace's next call, so
        # the ones that other calls follow come to the host
        h, ws = s["graph"], s["ws"]
        host = s["flags"] & ~tpg.TPG_OUT_DEVICE
        comp, _, arcs = tpg.ccfg(h, ws=ws)
        extracted = tpg.scc_paths(h, ws=ws, flags=host)
        internal = tpg.scc_internal_pps(h, ws=ws, flags=host)
        merged = tpg.merged_pps(h, ws=ws, flags=s["flags"])
        return {"comp": comp, "arcs": arcs, "extracted": [_arrays(x, ws) for x in extracted],
                "internal": _arrays(internal, ws), "merged": [_arrays(x, ws) for x in merged]}
    pred = sizer.predict(s["mlp"], s["graphs"]) if "mlp" in s else None
    r, _ = tpg.batch_test_paths(s["graphs"], ws=s["ws"], flags=s["flags"], predicted=pred)
    return {"pred": pred, "pp": _arrays(r.pp, s["ws"]), "tp": _arrays(r.tp, s["ws"]),
            "first": (r.pp_first, r.tp_first)}


def _joined(sets):
    return (np.concatenate([p.offsets for p in sets]), np.concatenate([p.vertices for p in sets]))


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

@functools.lru_cache(maxsize=64)
def _work(items):
    case = dict(items)
    if case["kind"] == "grad":
        n, io = case["rows"], tpg.MLP_IN + tpg.MLP_OUT
        mats = 32 * 128 + 128 * 128 + 128 * 65
        # products: forward, weight gradients, and the two hidden layers' gradients
        return 4 * (n * io + 2 * tpg.MLP.num_params()), 2 * n * (3 * mats - 32 * 128)
    s = prepare(case, 0)
    # every path returned is written once, with its offset; the graph is read
    return 4 * _outputs(run(s)) + 8 * 4 * 100, 0


def _outputs(r):
    """32-bit words of a result."""
    if r is None:
        return 0
    if isinstance(r, dict):
        return sum(_outputs(x) for x in r.values())
    if isinstance(r, (list, tuple)):
        return sum(_outputs(x) for x in r)
    n = r.numel() if hasattr(r, "numel") else r.size
    return n * (r.element_size() if hasattr(r, "numel") else r.itemsize) // 4


def work(case):
    b, f = _work(tuple(sorted((k, v) for k, v in case.items() if k != "name")))
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# The size predictor in 64 bits (path sets are whole numbers)
# ---------------------------------------------------------------------------

def _layers(p):
    out, q = [], 0
    for a, b in ((32, 128), (128, 128), (128, 65)):
        out.append((p[q:q + a * b].reshape(a, b).astype(np.float64),
                    p[q + a * b:q + a * b + b].astype(np.float64)))
        q += a * b + b
    return out


def _network(p, mean, std, x):
    (w1, b1), (w2, b2), (w3, b3) = _layers(p)
    xn = (x.astype(np.float64) - mean) / std
    h1 = np.maximum(xn @ w1 + b1, 0.0)
    h2 = np.maximum(h1 @ w2 + b2, 0.0)
    return xn, h1, h2, h2 @ w3 + b3


def exact(case, seed):
    if case["kind"] == "grad":
        x, t, p, mean, std = _predictor_inputs(case, seed)
        xn, h1, h2, y = _network(p, mean, std, x)
        (_, _), (w2, _), (w3, _) = _layers(p)
        e = y - t
        dy = 2.0 * e / e.size
        d2 = (dy @ w3.T) * (h2 > 0)
        d1 = (d2 @ w2.T) * (h1 > 0)
        g = [xn.T @ d1, d1.sum(0), h1.T @ d2, d2.sum(0), h2.T @ dy, dy.sum(0)]
        return {"grad": np.concatenate([v.reshape(-1) for v in g]), "loss": np.mean(e * e)}
    if case["kind"] == "batch" and case["learned"]:
        rng = np.random.default_rng(seed)
        x = tpg.features([tpg.load_cfg(_renumbered(g, sib, rng))
                          for g, sib in _members(case["base"], case["count"])])
        raw = np.fromfile(os.path.abspath(sizer.DEFAULT_MODEL), np.float32, offset=12)
        y = _network(raw[64:], raw[:32].astype(np.float64), raw[32:64].astype(np.float64), x)[3]
        return {"pred": y, "pp": (None, None), "tp": (None, None), "first": (None, None)}
    return None
