"""Graphs with straight lines (chains), which the path tree takes as single
vertices: chains that wrap around a ring, cycles that start inside a chain,
chains whose ids are neither neighbours nor ascending, one chain only, and
sizes around the rotation step (16 Ki leaves of one root) and the writer's
staged form (2048 vertices).  Prime paths, test paths and the path counts of
every length against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import check_tp, first_diff, same, say, ws

pytestmark = pytest.mark.gpu

S = ("stmt",)


def _diamond():
    return ("if", [S], [S], False)


def _subdivided(seed):
    """A random digraph with 0 to 4 vertices put on every arc, ids shuffled."""
    rng = np.random.default_rng(seed)
    base = cfggen.random_digraph(seed, int(rng.integers(1, 7)), 0.35)
    n, edges = base.n, []
    for a, b in base.edges():
        k = int(rng.integers(0, 5))
        stops = [a] + list(range(n, n + k)) + [b]
        n += k
        edges += list(zip(stops[:-1], stops[1:]))
    return cfggen.relabel(cfggen.from_edges(n, edges), rng.permutation(n), f"sub{seed}")


def _shuffled(g, seed):
    """Inner vertices renumbered at random."""
    perm = np.arange(g.n)
    perm[1:g.n - 1] = 1 + np.random.default_rng(seed).permutation(g.n - 2)
    return cfggen.relabel(g, perm, f"{g.name}_p{seed}")


def _check_any(g, flags):
    """Prime paths, cycles and path counts by length of any digraph."""
    h = tpg.load_cfg(g, tpg.TPG_LOAD_ANY_DIGRAPH)
    levels = np.zeros(g.n + 4, np.int64)
    pp, st = tpg.prime_paths(h, ws=ws(), flags=flags, level_counts=levels)
    ref, rst = oracle.prime_paths_local(g, 0, g.n)[:2]
    _, lv, cy = oracle.count(g)
    assert same(pp, ref), f"{g.name}: {first_diff(pp, ref)}"
    want = np.zeros(g.n + 4, np.int64)
    want[:g.n + 2] = lv + cy
    assert np.array_equal(levels, want), g.name
    assert st["n_cycles"] == int(cy.sum()) and st["n_pp"] == len(ref)
    assert st["n_nodes"] == int(want.sum()) and st["n_extensions"] == int(want[2:].sum())
    assert st["n_levels"] == int(np.nonzero(want)[0].max())
    assert st["peak_level_nodes"] == int(want.max())


@pytest.mark.parametrize("flags", [0, tpg.TPG_FORCE_TWO_PASS])
def test_rings_lines_and_subdivided_digraphs(flags):
    for n in (1, 2, 3, 63, 64, 65, 130):
        say("case ring and line", n, flags)
        _check_any(cfggen.cycle_graph(n), flags)
        _check_any(_shuffled(cfggen.cycle_graph(n), n), flags)
        _check_any(cfggen.path_graph(n), flags)
    for seed in range(60):
        say("case subdivided", seed, flags)
        _check_any(_subdivided(seed), flags)


@pytest.mark.parametrize("k", [3, 13])
@pytest.mark.parametrize("seed", [0, 1])
def test_cycles_from_inside_a_chain(k, seed):
    """A loop whose body opens with a chain of three: with 13 diamonds behind
    it that chain's root has over 16 Ki leaves."""
    body = [S, S] + [_diamond() for _ in range(k)] + [("if", [S], [S], True), S]
    g = cfggen.lower_program([S, ("while", body), S], name=f"chainloop{k}")
    say("case chain loop", k, seed)
    check_tp(_shuffled(g, seed) if seed else g, local=True)


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4096])
def test_long_lines(n):
    """Straight lines around one loop, n vertices in all."""
    loop = ("while", [_diamond(), S, S])
    rest = n - cfggen.lower_program([loop]).n
    g = cfggen.lower_program([S] * (rest // 2) + [loop] + [S] * (rest - rest // 2), name=f"line{n}")
    assert g.n == n
    say("case long line", n)
    check_tp(g, local=True)


@pytest.mark.parametrize("chunk", [1, 5, 32])
def test_streamed_ranges_cut_chains(chunk):
    """Ranges of first vertices that cut chains: the chunks concatenate to
    the canonical set and the totals stay those of the whole graph."""
    body = [S, S, S, _diamond(), S, ("if", [S, S], [S], True), S, S]
    g = _shuffled(cfggen.lower_program([S, S, ("while", body), S, S, S], name="cut"), 3)
    h = tpg.load_cfg(g)
    ref, rst = oracle.prime_paths_local(g, 0, g.n)[:2]
    parts = []
    say("case streamed chains", chunk)
    tot, st = tpg.prime_paths_stream(h, lambda c, a, b: parts.append((c, a, b)), ws=ws(),
                                     chunk_vertices=chunk)
    assert np.array_equal(np.concatenate([c.vertices for c, _, _ in parts]), ref.vertices)
    assert tot.digest == oracle.digest(ref)
    for c, a, b in parts:
        firsts = c.vertices[c.offsets[:-1]]
        assert ((firsts >= a) & (firsts < b)).all()
    assert st["n_cycles"] == rst["n_cycles"] and st["n_extensions"] == rst["n_extensions"]


def _hub(fan, seed):
    """A switch of `fan` arms in a loop, with arcs between arms and back to
    the switch from some of them (arcs off the BFS tree at every slot)."""
    rng = np.random.default_rng(seed)
    edges = [(0, 1)]
    for k in range(fan):
        edges += [(1, 2 + k), (2 + k, 2 + fan)]
        if rng.random() < 0.3:
            edges.append((2 + k, 1))
        if rng.random() < 0.1:
            edges.append((2 + k, 2 + int(rng.integers(0, fan))))
    edges += [(2 + fan, 1), (2 + fan, 3 + fan)] if fan < 64 else [(2 + fan, 3 + fan)]
    return cfggen.from_edges(4 + fan, edges, 0, 3 + fan, f"hub{fan}_{seed}")


@pytest.mark.parametrize("fan", [2, 5, 33, 63, 64])
def test_test_path_order_with_many_arcs(fan):
    """Test paths in order where one vertex has up to 64 arcs off the BFS
    tree, alone, with ids shuffled, and as a union of graphs."""
    graphs = []
    for seed in range(3):
        g = _hub(fan, seed)
        say("case hub", fan, seed)
        check_tp(g, local=True)
        check_tp(_shuffled(g, seed + 1), local=True)
        graphs.append(g)
    for seed in range(6):
        graphs.append(cfggen.random_small_cfg(900 + 10 * fan + seed, 8 + 3 * seed, extra=4 + 2 * seed))
        say("case dense", fan, seed)
        check_tp(graphs[-1], local=True)
    res, _ = tpg.batch_test_paths([tpg.load_cfg(g) for g in graphs], ws=ws())
    for i, g in enumerate(graphs):
        rp = oracle.prime_paths_local(g, 0, g.n)[0]
        rt = oracle.test_paths(g, rp)[0]
        (po, pv), (to, tv) = res.graph(i)
        assert np.array_equal(po, rp.offsets) and np.array_equal(pv, rp.vertices), g.name
        assert np.array_equal(to, rt.offsets) and np.array_equal(tv, rt.vertices), g.name


def _two_level_switch(a, b):
    """A switch of a arms, each a switch of b arms, some with a way back to
    their own switch: 2 + a (b + 1) + 1 chains."""
    edges, n = [], 2 + a * (b + 1) + 1
    for i in range(a):
        v = 2 + i * (b + 1)
        edges.append((1, v))
        for j in range(1, b + 1):
            edges += [(v, v + j), (v + j, n - 1)]
            if (i + j) % 3 == 0:
                edges.append((v + j, v))
    return cfggen.from_edges(n, [(0, 1)] + edges, 0, n - 1, f"switch{a}x{b}")


def _layers(a, b):
    """entry -> a vertices -> each of b vertices -> exit."""
    n = 2 + a + b
    edges = [(0, 1 + i) for i in range(a)] + [(1 + a + j, n - 1) for j in range(b)]
    edges += [(1 + i, 1 + a + j) for i in range(a) for j in range(b)]
    return cfggen.from_edges(n, edges, 0, n - 1, f"layers{a}x{b}")


@pytest.mark.parametrize("name", ["switch25x9", "switch30x9", "switch60x30", "layers20x20", "layers60x60"])
def test_shortest_paths_at_the_kernel_sizes(name):
    """BFS trees of at most and of more than 256 chains, and graphs on both
    sides of the staged size."""
    a, b = (int(x) for x in name.lstrip("switchlayers").split("x"))
    g = _two_level_switch(a, b) if name.startswith("switch") else _layers(a, b)
    say("case", name, g.n)
    check_tp(g, local=True)
    check_tp(_shuffled(g, 5), local=True)
