"""Cooperative merges (merge_min) on graphs without dense rows: windows whose
partial matches share both lists of the leaf, and windows that do not.  Counts
equal the oracle's."""
import numpy as np
import pytest

import oracle
import xmgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xa():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_11105_amd as xa
    return xa


@pytest.mark.parametrize("merge_min", [4, 64])
def test_two_partial_matches_with_the_same_lists(xa, merge_min):
    """4-cycle: z -> y1 -> x, z -> y2 -> x, x -> w_i, w_i -> z; the window of root
    x holds (x, y1, z) and (x, y2, z), whose leaves are the same 100 nodes."""
    z, y1, y2, x = range(4)
    w = np.arange(4, 104)
    src = np.concatenate([[z, y1, z, y2], np.full(100, x), w])
    dst = np.concatenate([[y1, x, y2, x], w, np.full(100, z)])
    g = xmgen.from_arcs(104, src, dst)
    p = xmgen.named("c4")
    G = xa.Graph(g, dense_rows=0)
    assert oracle.count(g, p) == 800
    assert xa.count(G, [xa.Plan(p, graph=G)], merge_min=merge_min, chunk=1) == [800]


@pytest.mark.parametrize("n, deg", [(60, 30), (300, 20), (300, 90)])
@pytest.mark.parametrize("opts", [dict(merge_min=4), dict(merge_min=64), dict(merge_min=8, chunk=1),
                                  dict(merge_min=8, merge_ratio=1, cap=64, split=64, waves_per_cu=4)])
def test_merges_with_and_without_shared_lists(xa, n, deg, opts):
    rng = np.random.default_rng(n + deg)
    u, v = rng.integers(0, n, (2, n * deg))
    g = xmgen.from_arcs(n, u, v)
    P = xmgen.Pattern
    pats = [xmgen.named(q) for q in ("ffl", "c3", "c4", "bifan")]
    # the leaf is next to the first two vertices only, the vertex before it is not
    pats.append(P(4, ((0, 1), (0, 2), (1, 2), (0, 3), (1, 3))))
    want = [oracle.count(g, p) for p in pats]
    G = xa.Graph(g, dense_rows=0)
    print("[case]", n, deg, opts, flush=True)
    for p, w in zip(pats, want):
        for reduced in (True, False):
            assert xa.count(G, [xa.Plan(p, reduced=reduced, graph=G)], **opts) == [w]
    # one launch of one-leaf plans
    assert xa.count(G, [xa.Plan(p, reduced=False, graph=G) for p in pats], **opts) == want
    assert xa.count(G, [xa.Plan(p, reduced=False, graph=G, symmetry="above") for p in pats], **opts) == want
