"""Base lists scanned one by one by a whole wave: list lengths at the edges of
its steps (one, two and four tiles of 64 elements, and remainders), with dense
rows, with sorted-list searches and with both among one parent's probes.
Counts are whole numbers and equal the oracle's."""
import numpy as np
import pytest

import oracle
import xmgen

pytestmark = pytest.mark.gpu

LENGTHS = [1, 31, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 320, 321, 449, 512, 513]


def lists_graph(seed=7, n=1301):
    """Node i's out-list has LENGTHS[i] random nodes, node 40 + i's in-list
    too, and arcs among the first 90 nodes close many small patterns."""
    rng = np.random.default_rng(seed)
    src, dst = [], []
    for i, ln in enumerate(LENGTHS):
        to = rng.choice(np.arange(90, n), ln, replace=False)
        src += [np.full(ln, i), to]
        dst += [to, np.full(ln, 40 + i)]
    core = rng.random((90, 90)) < 0.3
    u, v = np.nonzero(core)
    extra = rng.integers(0, n, (2, 2000))
    return xmgen.from_arcs(n, np.concatenate(src + [u, extra[0]]), np.concatenate(dst + [v, extra[1]]))


@pytest.fixture(scope="module")
def xa():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_11105_amd as xa
    return xa


@pytest.fixture(scope="module")
def case():
    g = lists_graph()
    pats = [xmgen.named(p) for p in ("ffl", "c3", "bifan", "c4")]
    return g, pats, [oracle.count(g, p) for p in pats]


@pytest.mark.parametrize("rows", [dict(dense_rows=0), dict(row_min=32), dict(row_min=200)])
@pytest.mark.parametrize("opts", [dict(), dict(cap=64, split=64), dict(cap=200, split=128, waves_per_cu=4)])
def test_lists_at_step_edges(xa, case, rows, opts):
    g, pats, want = case
    print("[case]", rows, opts, flush=True)
    G = xa.Graph(g, **rows)
    for reduced in (True, False):
        assert xa.count(G, [xa.Plan(p, reduced=reduced, graph=G) for p in pats], **opts) == want
    sym = [xa.Plan(p, graph=G, symmetry=s) for p in pats for s in ("above", "below")]
    assert xa.count(G, sym, **opts) == [w for w in want for _ in range(2)]


@pytest.mark.parametrize("rows", [dict(dense_rows=0), dict(row_min=64)])
def test_several_probes_per_parent(xa, rows):
    """Four mutually joined vertices plus a leaf: up to three probes a test."""
    rng = np.random.default_rng(3)
    n = 400
    u, v = np.nonzero(rng.random((n, n)) < 0.2)
    g = xmgen.from_arcs(n, u, v)
    pats = [xmgen.Pattern(4, ((0, 1), (0, 2), (0, 3), (1, 2), (1, 3), (2, 3))),
            xmgen.Pattern(4, ((0, 1), (1, 0), (0, 2), (1, 2), (3, 0), (3, 1), (2, 3)))]
    G = xa.Graph(g, **rows)
    for reduced in (True, False):
        assert xa.count(G, [xa.Plan(p, reduced=reduced, graph=G) for p in pats]) == [oracle.count(g, p) for p in pats]


def skewed_graph(seed=11, n=20011):
    """14 nodes with out- and in-lists of 130 to 4,000 nodes, most at low ids
    (rows with dense heads of one to three chunks of 256 words, the last words
    of a row in none), joined to each other, over a sparse background."""
    rng = np.random.default_rng(seed)
    src, dst = [], []
    for i, ln in enumerate([130, 257, 500, 511, 512, 700, 1000, 1500, 2000, 2500, 3000, 3500, 3999, 4000]):
        for into in (False, True):
            x = np.unique((n * rng.random(2 * ln) ** (1.0 + 0.5 * (i % 4))).astype(np.int64))
            x = np.concatenate([rng.choice(x, min(ln, x.size), replace=False), np.arange(n - 3, n)])
            h = np.full(x.size, i)
            src.append(x if into else h)
            dst.append(h if into else x)
    u, v = np.nonzero(rng.random((14, 14)) < 0.6)
    e = rng.integers(0, n, (2, 30000))
    return xmgen.from_arcs(n, np.concatenate(src + [u, e[0]]), np.concatenate(dst + [v, e[1]]))


def test_dense_heads(xa):
    g = skewed_graph()
    P = xmgen.Pattern
    pats = [xmgen.named("ffl"), xmgen.named("c3"), P(4, ((0, 1), (0, 2), (1, 2), (0, 3), (1, 3))),
            P(4, ((0, 1), (1, 0), (0, 2), (2, 1), (3, 0), (1, 3)))]
    want = [oracle.count(g, p) for p in pats]
    for rows in (dict(row_min=64), dict(row_min=64, dense_rows=24 * 2504), dict(dense_rows=0)):
        G = xa.Graph(g, **rows)
        print("[case]", G.dense_rows_info(), flush=True)
        for reduced in (True, False):
            assert xa.count(G, [xa.Plan(p, reduced=reduced, graph=G) for p in pats]) == want
        sym = [xa.Plan(p, graph=G, symmetry=s, reduced=r) for p in pats for s in ("above", "below") for r in (True, False)]
        assert xa.count(G, sym) == [w for w in want for _ in range(4)]


@pytest.mark.parametrize("reduced", [True, False])
def test_one_heavy_root_is_shared_out(xa, reduced):
    """One hub root whose whole work is a single task (its first-level list is
    not split): other waves get parts of its windows, as single parents and as
    id ranges below one parent, and the counts stay the root's."""
    g = xmgen.rmat(13, seed=3)
    hub = np.array([int(np.argmax(g.out_deg() + g.in_deg()))], dtype=np.uint32)
    G = xa.Graph(g)
    for name in ("ffl", "c4", "bifan"):
        p = xmgen.named(name)
        plan = xa.Plan(p, reduced=reduced, graph=G, root_vertex=0)
        want = oracle.count(g, p, roots=hub, root_vertex=0)
        for opts in (dict(split=4096, split_work=1 << 30), dict(split=4096, split_work=1 << 30, cap=4096, chunk=1)):
            print("[case]", name, reduced, opts, flush=True)
            assert xa.count(G, [plan], roots=hub, **opts) == [want]


@pytest.mark.parametrize("n", [63, 8192, 8193, 65536, 65537, 150001])
def test_short_lists_against_a_shared_list(xa, n):
    """Short lists tested against a bit map of a list that a window shares: id
    ranges at the map's sizes (every id its own bit, or ids that share bits),
    kept and refilled between windows and plans, with one and with two leaves,
    and with too little LDS for the whole map."""
    rng = np.random.default_rng(n)
    m = 6 * n
    u, v = rng.integers(0, n, (2, m))
    # some arcs between ids that share low bits, and triangles to find
    w = (u[: m // 8] + 32768 * rng.integers(0, 4, m // 8)) % n
    src = np.concatenate([u, v[: m // 8], u[: m // 8]])
    dst = np.concatenate([v, w, w])
    g = xmgen.from_arcs(n, src, dst)
    P = xmgen.Pattern
    pats = [xmgen.named("ffl"), xmgen.named("c3"), xmgen.named("c4"), xmgen.named("c5chord"),
            P(4, ((0, 1), (0, 2), (1, 2), (0, 3), (1, 3)))]
    want = [oracle.count(g, p) for p in pats]
    G = xa.Graph(g)
    for opts in (dict(), dict(waves_per_cu=4), dict(waves_per_cu=12), dict(waves_per_cu=16), dict(cap=64, split=64)):
        print("[case]", n, opts, flush=True)
        for reduced in (True, False):
            assert xa.count(G, [xa.Plan(p, reduced=reduced, graph=G) for p in pats], **opts) == want
        assert xa.count(G, [xa.Plan(p, graph=G, symmetry="above") for p in pats[:3]], **opts) == want[:3]


@pytest.mark.parametrize("n, deg", [(40, 12), (300, 20), (300, 90)])
def test_sets_shared_by_a_whole_window(xa, n, deg):
    """Leaf groups with a leaf whose neighbours are bound early, so windows of
    partial matches share its candidate set (measured once): windows smaller
    than a wave, cut by slices, and sets below and above the scan lengths.  The
    last pattern has one leaf, next to a plan with several in the same launch."""
    rng = np.random.default_rng(n + deg)
    u, v = rng.integers(0, n, (2, n * deg))
    g = xmgen.from_arcs(n, u, v)
    P = xmgen.Pattern
    pats = [xmgen.named("tt4p"), P(4, ((0, 1), (0, 2), (1, 2), (3, 0), (3, 1))),
            P(5, ((0, 1), (1, 2), (0, 3), (1, 3), (1, 4), (4, 0), (2, 0))) if deg < 100 else xmgen.named("c4"),
            P(4, ((0, 1), (1, 2), (2, 3), (3, 1)))]
    want = [oracle.count(g, p) for p in pats]
    G = xa.Graph(g, row_min=64)
    for opts in (dict(), dict(cap=64, split=64), dict(cap=100, split=64, waves_per_cu=4)):
        print("[case]", n, deg, opts, flush=True)
        assert xa.count(G, [xa.Plan(p, graph=G) for p in pats], **opts) == want
        for p, w in zip(pats, want):
            assert xa.count(G, [xa.Plan(p, graph=G)], **opts) == [w]
            assert xa.count(G, [xa.Plan(p, graph=G, symmetry="below")], **opts) == [w]
