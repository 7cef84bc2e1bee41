"""Donated work: launches whose whole work starts as one task.  The donated-task
counter of the launch's own workspace shows that tasks were handed out, and the
counts stay those of the oracle or of another plan of the same pattern."""
import os
import re

import numpy as np
import pytest

import oracle
import xmgen

pytestmark = pytest.mark.gpu
ONE_TASK = dict(split=4096, split_work=1 << 30)  # a root of up to 4,096 first-level candidates stays whole


def constant(name):
    """The value of a constant or control word in the launch interface's header."""
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2404_11105_amd", "csrc",
                        "kernels.h")
    text = re.search(name + r" = (?:(\d+)u << )?(\d+)[,;]", open(path).read())
    return int(text.group(1)) << int(text.group(2)) if text.group(1) else int(text.group(2))


@pytest.fixture(scope="module")
def xa():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2404_11105_amd as xa
    return xa


def hub_of(g):
    return np.array([int(np.argmax(g.out_deg() + g.in_deg()))], dtype=np.uint32)


def run(xa, G, plan, roots, **opts):
    """Counts, and how many tasks were donated (the queue's tail, in the control words
    at the start of the workspace)."""
    import torch
    c = xa.Counter(G, [plan], roots=roots, **opts)
    c.run()
    counts, status = c.results()
    assert status == [0]
    return counts[0], int(c.workspace.view(torch.int32)[constant("kCtlDonTail")])


def test_id_ranges_of_a_leaf_pass_are_handed_out(xa):
    """One level below the root: only ranges of a leaf window can be donated."""
    n = 4096
    rng = np.random.default_rng(5)
    u, v = np.nonzero(rng.random((n, n)) < 0.5)
    g = xmgen.from_arcs(n, u, v)
    G = xa.Graph(g, dense_rows=0)
    p = xmgen.named("ffl")
    plan = xa.Plan(p, reduced=False, graph=G, root_vertex=0)
    assert plan.describe()["e"] == 2
    root = np.array([7], dtype=np.uint32)
    want = oracle.count(g, p, roots=root, root_vertex=0)
    for opts in (dict(), dict(cap=8192), dict(waves_per_cu=4)):
        got, donated = run(xa, G, plan, root, **ONE_TASK, **opts)
        print("[case]", opts, "donated", donated, flush=True)
        assert got == want and donated > 0


@pytest.mark.parametrize("name", ["c4", "bifan"])
def test_parents_are_handed_out_between_short_leaf_windows(xa, name):
    """Leaf windows too short to be cut (under two looks long) must not keep the task
    from handing off parents: a few wide donations only would leave hundreds of
    waves idle."""
    g = xmgen.rmat(15, seed=2)
    G = xa.Graph(g)
    p = xmgen.named(name)
    plan = xa.Plan(p, reduced=False, graph=G, root_vertex=0)
    root = hub_of(g)
    want, _ = run(xa, G, xa.Plan(p, graph=G, root_vertex=0), root)
    got, donated = run(xa, G, plan, root, **ONE_TASK)
    print("[case]", name, "donated", donated, flush=True)
    assert got == want and donated > 1000


def test_slots_are_handed_out_again(xa):
    """More tasks than the queue has slots, and more than a launch had in all when
    each slot was used once; counted by another plan too."""
    g = xmgen.rmat(17, seed=1)
    G = xa.Graph(g)
    p = xmgen.named("c5chord")
    root = hub_of(g)
    want, _ = run(xa, G, xa.Plan(p, graph=G, root_vertex=0), root)
    got, donated = run(xa, G, xa.Plan(p, reduced=False, graph=G, root_vertex=0), root)
    print("[case] donated", donated, "slots", constant("kDonCap"), flush=True)
    assert got == want
    assert donated > constant("kDonCap") and donated > 1 << 18


def test_donated_ranges_list_every_embedding_once(xa):
    n = 2048
    rng = np.random.default_rng(6)
    u, v = np.nonzero(rng.random((n, n)) < 0.5)
    g = xmgen.from_arcs(n, u, v)
    G = xa.Graph(g, dense_rows=0)
    p = xmgen.named("ffl")
    plan = xa.Plan(p, reduced=False, graph=G, root_vertex=0)
    root = np.array([7], dtype=np.uint32)
    want = oracle.count(g, p, roots=root, root_vertex=0)
    got, donated = run(xa, G, plan, root, **ONE_TASK, list_cap=want)
    print("[case] listing, donated", donated, flush=True)
    c = xa.Counter(G, [plan], roots=root, list_cap=want, **ONE_TASK)
    c.run()
    found, rows = c.listed()
    rows = rows.astype(np.int64)
    assert got == found == want and donated > 0
    assert (rows[:, 0] == 7).all() and np.unique(rows[:, 1] * n + rows[:, 2]).size == want


def test_donation_on_the_static_array(xa):
    from tests.test_zz_no_alloc import static_count
    g = xmgen.rmat(15, seed=2)
    G = xa.Graph(g)
    c = xa.Counter(G, [xa.Plan(xmgen.named("c5chord"), graph=G, root_vertex=0)], roots=hub_of(g))
    c.run()
    want = c.results()[0]
    plan = xa.Plan(xmgen.named("c5chord"), reduced=False, graph=G, root_vertex=0)
    for _ in range(2):
        got, status = static_count(xa, G, [plan], roots=c.roots, roots_host=c.roots_host)
        assert status == [0] and got == want
