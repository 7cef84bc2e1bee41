"""The default number of waves, read from the workspace it needs, and the counts
of launches on each side of the rule."""
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


@pytest.mark.parametrize("n, deg, names, share, waves", [
    (3001, 4, "ffl,c4", 0, 12), (300007, 4, "ffl,c4", 0, 12), (466100, 24, "ffl", 0, 12), (466000, 24, "c4", 0, 12),
    (466100, 24, "c4", 0, 24), (466100, 24, "c4", 1, 12)])
def test_graphs_without_long_lists(xa, n, deg, names, share, waves):
    """Little to do: 12 waves per CU, whose kernel tests short lists against a bit map
    in LDS.  Plans of several levels with 2^28 or more 2-paths: 24."""
    g = xmgen.uniform_digraph(n, deg * n, 1)
    pats = [xmgen.named(p) for p in names.split(",")]
    G = xa.Graph(g)
    assert max(G.info()["max_out"], G.info()["max_in"]) <= 64
    plans = [xa.Plan(p, graph=G, root_share=share) for p in pats]
    print("[case]", n, deg, names, share, flush=True)
    assert xa.api.workspace_bytes(G, plans) == xa.api.workspace_bytes(G, plans, waves_per_cu=waves)
    assert xa.api.workspace_bytes(G, plans, waves_per_cu=12) != xa.api.workspace_bytes(G, plans, waves_per_cu=24)
    got = xa.count(G, plans)
    if deg < 10:
        assert got == [oracle.count(g, p) for p in pats]
    assert got == xa.count(G, plans, waves_per_cu=12) == xa.count(G, plans, waves_per_cu=24, chunk=1)


@pytest.mark.parametrize("names, waves", [("path3", 12), ("arc,outstar3,mixed_star", 12), ("path3,ffl", 24)])
def test_plans_without_levels_below_the_root(xa, names, waves):
    g = xmgen.rmat(12, seed=5)
    pats = [xmgen.named(p) for p in names.split(",")]
    G = xa.Graph(g)
    plans = [xa.Plan(p, graph=G) for p in pats]
    print("[case]", names, flush=True)
    assert xa.api.workspace_bytes(G, plans) == xa.api.workspace_bytes(G, plans, waves_per_cu=waves)
    assert xa.api.workspace_bytes(G, plans, waves_per_cu=12) != xa.api.workspace_bytes(G, plans, waves_per_cu=24)
    want = [oracle.count(g, p) if p.k < 4 else None for p in pats]
    got = xa.count(G, plans)
    assert all(w is None or w == c for w, c in zip(want, got))
    assert got == xa.count(G, plans, waves_per_cu=24) == xa.count(G, plans, waves_per_cu=4)


@pytest.mark.parametrize("waves", [0, 12, 24])
def test_listing_and_merging_launches(xa, waves):
    """They run the kernel of 12 waves per CU, whatever is asked for, and by default
    no more are reserved.  Every embedding is listed, and counts are the oracle's."""
    import torch
    g = xmgen.rmat(11, seed=4)
    p = xmgen.named("ffl")
    want = oracle.count(g, p)
    G = xa.Graph(g)
    plan = xa.Plan(p, reduced=False, graph=G)
    rows = torch.empty(3 * 16, dtype=torch.int32, device=G.device)
    n = torch.zeros(1, dtype=torch.int64, device=G.device)
    for opts in (dict(listing=(rows, 16, n)), dict(merge_min=64)):
        used = xa.api.workspace_bytes(G, [plan], waves_per_cu=waves, **opts)
        assert used == xa.api.workspace_bytes(G, [plan], waves_per_cu=waves or 12, **opts)
    print("[case]", waves, flush=True)
    found, listed = xa.list_embeddings(G, p, cap=want, waves_per_cu=waves)
    assert found == want and len({tuple(r) for r in listed.tolist()}) == want
    G = xa.Graph(g, dense_rows=0)
    assert xa.count(G, [xa.Plan(p, reduced=False, graph=G)], merge_min=16, waves_per_cu=waves) == [want]


def test_more_waves_than_can_be_resident(xa):
    """Asked for more waves than the kernel's registers allow: nothing is reserved
    for the rest, and the autotuner does not try them."""
    import torch
    from paper_2404_11105_amd import tune
    g = xmgen.rmat(11, seed=4)
    p = xmgen.named("ffl")
    G = xa.Graph(g)
    plan = xa.Plan(p, reduced=False, graph=G)
    size = xa.api.workspace_bytes
    assert size(G, [plan], waves_per_cu=32) == size(G, [plan], waves_per_cu=24)
    rows = torch.empty(3 * 16, dtype=torch.int32, device=G.device)
    n = torch.zeros(1, dtype=torch.int64, device=G.device)
    for opts in (dict(listing=(rows, 16, n)), dict(merge_min=64)):
        assert size(G, [plan], waves_per_cu=24, **opts) == size(G, [plan], waves_per_cu=12, **opts)
    assert max(dict(tune.SPACE)["waves_per_cu"]) == 24
    want = oracle.count(g, p)
    for waves in (24, 32):
        assert xa.count(G, [plan], waves_per_cu=waves) == [want]
