"""Deep graphs of many chains, where the search for shortest paths has as many
levels as vertices and the exit as many predecessors, on both sides of its
sizes (256 and 1024 chains, 64 predecessors), and shortest paths that tie after
long ways apart."""
import time

import pytest

import oracle
from paper_2210_16998_amd import cfggen, tpg
from tests.gpu_util import check_tp, say, ws
from tests.test_gpu_narrow import _fans

pytestmark = pytest.mark.gpu


def _looped(g, v):
    """g with an arc from v to itself: its test paths are not its prime paths."""
    return cfggen.from_edges(g.n, sorted(g.edges() + [(v, v)]), name=g.name + "_looped")


def _guards(n, flip=False):
    """n vertices in a row, each of which may leave to the exit; flip: with the
    inner ones numbered from the end."""
    order = [0] + (list(range(n - 2, 0, -1)) if flip else list(range(1, n - 1))) + [n - 1]
    edges = set(zip(order, order[1:])) | {(v, n - 1) for v in order[:-1]}
    return cfggen.from_edges(n, sorted(edges), name=f"guards_{n}_{flip}")


def _switches(a, b):
    """A switch of switches, all of whose leaves go to the exit."""
    n = 2 + a + a * b
    edges = [(0, 1 + i) for i in range(a)]
    for i in range(a):
        for x in range(1 + a + i * b, 1 + a + (i + 1) * b):
            edges += [(1 + i, x), (x, n - 1)]
    return cfggen.from_edges(n, edges, name=f"switches_{a}_{b}")


def _rails(length, fan, flip):
    """Two rails that part at the entry, each with exits all along, and fan out
    into as many equally long ways to the head of a loop: every pair of them is
    compared over the whole rails.  flip: the other rail's ways come first."""
    a = [1 + (2 * i if flip else i) for i in range(length)]
    b = [2 + 2 * i if flip else 1 + length + i for i in range(length)]
    fa = [1 + 2 * length + (2 * i + 1 if flip else 2 * i) for i in range(fan)]
    fb = [1 + 2 * length + (2 * i if flip else 2 * i + 1) for i in range(fan)]
    t, end = 1 + 2 * length + 2 * fan, 3 + 2 * length + 2 * fan
    edges = [(0, a[0]), (0, b[0]), (t, end), (t, t + 1), (t + 1, t)]
    for rail, f in ((a, fa), (b, fb)):
        edges += list(zip(rail, rail[1:])) + [(v, end) for v in rail]
        edges += [(rail[-1], v) for v in f] + [(v, t) for v in f]
    return cfggen.from_edges(end + 1, sorted(edges), name=f"rails_{length}_{fan}_{flip}")


@pytest.mark.parametrize("flip", [False, True])
@pytest.mark.parametrize("n", [3, 65, 66, 67, 255, 256, 257, 1023, 1024, 1025])
def test_early_exits(n, flip):
    say("case", n, flip)
    check_tp(_guards(n, flip), local=True)
    for v in {1, n // 2, n - 2}:
        check_tp(_looped(_guards(n, flip), v), local=True)


@pytest.mark.parametrize("a,b", [(8, 8), (13, 5), (5, 13), (15, 16), (31, 32), (33, 60)])
def test_switches_into_one_exit(a, b):
    say("case", a, b)
    check_tp(_switches(a, b), local=True)
    check_tp(_looped(_switches(a, b), a), local=True)
    check_tp(_looped(_switches(a, b), a + b // 2), local=True)


# levels of more than 2048 nodes, swept one or two to a launch: 16 successors and
# 17, and fewer; odd and even numbers of such levels
@pytest.mark.parametrize("widths", [(16, 16, 16), (17, 17, 8), (16, 16, 16, 3), (17, 3, 17, 17), (9, 9, 9, 4)])
@pytest.mark.parametrize("back", [False, True])
def test_wide_levels_by_successors(widths, back):
    if back:
        widths = widths[:3]  # and the loop's paths
    g, _ = _fans(widths, back)
    say("case", g.name, back)
    check_tp(g, local=True)
    if not back:
        check_tp(_looped(g, g.n // 2), local=True)


# fan 31: 63 predecessors, one thread's; 34: a wave's.  The thread's walks pass
# their limit from a length of about 25 on
@pytest.mark.parametrize("flip", [False, True])
@pytest.mark.parametrize("length,fan", [(4, 31), (40, 31), (40, 34), (120, 31), (420, 31)])
def test_ties_after_long_ways(length, fan, flip):
    say("case", length, fan, flip)
    check_tp(_rails(length, fan, flip), local=True)


def test_batch_of_deep_graphs():
    """Enough of them for a wave each, and with larger ones among them."""
    for sizes in ([30 + k for k in range(70)], [30 + k for k in range(8)] + [300, 1030]):
        gs = [_looped(_guards(n, bool(n & 1)), n // 2) for n in sizes] + [_rails(30, 31, True)]
        r, _ = tpg.batch_test_paths([tpg.load_cfg(g) for g in gs], ws=ws())
        for k, g in enumerate(gs):
            say("case", g.name)
            pp = oracle.prime_paths_local(g, 0, g.n)[0]
            for (off, vtx), want in zip(r.graph(k), (pp, oracle.test_paths(g, pp)[0])):
                assert (off == want.offsets).all() and (vtx == want.vertices).all(), g.name


def test_deep_graph_costs_no_pass_per_level():
    """1000 early exits: with the test paths a call takes about what the prime
    paths alone take (6.3 times that when every level looked at all arcs)."""
    h = tpg.load_cfg(_looped(_guards(1000), 500))
    flags = tpg.TPG_NO_TIMING | tpg.TPG_OUT_DEVICE

    def ms(f):
        t = []
        for _ in range(5):
            t0 = time.perf_counter()
            f(h, ws=ws(), flags=flags)
            t.append(time.perf_counter() - t0)
        return 1e3 * min(t)
    pp, tp = ms(tpg.prime_paths), ms(tpg.test_paths)
    say("prime paths", pp, "ms, test paths", tp, "ms")
    assert tp < 2.0 * pp


# narrow levels by the words of their sets: 2048 nodes up to 8 words, 1024 at 16,
# 512 at 32, 256 at 64 words
@pytest.mark.parametrize("widths,exits", [((44, 46), 280), ((31, 33), 600), ((22, 23), 1400), ((15, 17), 2100)])
def test_narrow_levels_by_words(widths, exits):
    """Fans and, from the entry, a row of vertices that may all leave to the
    exit: levels of the row's length and fewer, and more where the fans end."""
    g, _ = _fans(widths)
    n, end = g.n, g.n + exits
    edges = g.edges() + [(n - 1, end), (0, n)] + [(v, v + 1) for v in range(n, end)]
    edges = sorted(set(edges) | {(v, end) for v in range(n, end)})
    g = cfggen.from_edges(end + 1, edges, name=f"{g.name}_{exits}")
    say("case", g.name, g.n)
    check_tp(g, local=True)
    check_tp(_looped(g, 3), local=True)
