"""Measured cases of the counting path, from the smallest call to the batch.

Each case is one call (or one burst of requests) that a program using this
package makes, on a seeded synthetic graph of a size the package's own
benchmark and tests use, or near one.  A case's fields:

  graph     "uniform" (n nodes, m arcs) or "rmat" (2**scale nodes, 16 draws a
            node, cut to the first n nodes when n is given)
  order     "generated" ids, "degree" (ranked by the library at load) or
            "ranked" (ranked by the program before loading device arrays)
  patterns  names, or "pool:P" = the first P stored patterns of each size 3-6
            with their root shares, or "serve:R" = R requests of the serving pool
  call      how the program calls: count / run / replay / subset / anchored /
            list / serve
"""
import numpy as np
import torch

import xmgen
from paper_2404_11105_amd import Counter, Graph, Plan, count, count_anchored, workloads
from paper_2404_11105_amd.serve import GpuBackend, Server

MOTIFS = "ffl,c3,bifan,c4"


def listed():
    return [
        # the smallest call: one pattern on a small graph, asked once; launches,
        # allocations and the wait for the answer are all of it
        {"name": "uniform2k_count", "graph": "uniform", "n": 2000, "m": 20000, "patterns": "bifan", "call": "count"},
        # the same size in a loop that captured its launch once
        {"name": "uniform2k_replay", "graph": "uniform", "n": 2000, "m": 20000, "patterns": MOTIFS, "call": "replay"},
        # short lists only (no node has a dense row), an odd node count, 4- and
        # 5-vertex patterns without symmetry breaking
        {"name": "uniform30k_run", "graph": "uniform", "n": 30011, "m": 600007, "patterns": "c4,tt4p,c5chord",
         "call": "run"},
        # a pattern anchored at given nodes: one small launch a node
        {"name": "anchored_rmat18", "graph": "rmat", "scale": 18, "patterns": "ffl", "vertex": 0, "nodes": 8,
         "call": "anchored"},
        # a tenth of the start nodes (the share-of-start-nodes workload)
        {"name": "subset_rmat16", "graph": "rmat", "scale": 16, "patterns": MOTIFS, "vertex": 0, "percent": 10,
         "call": "subset"},
        # the four motifs, symmetry broken, graph in degree order, captured
        {"name": "motifs_rmat16_replay", "graph": "rmat", "scale": 16, "order": "degree",
         "patterns": "ffl,c3:above,bifan:below,c4:above", "call": "replay"},
        # the same motifs as they come: generated order, unreduced plans, a
        # node count that is no power of two
        {"name": "motifs_rmat16_unreduced", "graph": "rmat", "scale": 16, "n": 60001, "patterns": MOTIFS,
         "unreduced": True, "call": "run"},
        # every embedding written out, then put in one order (the rows come in none)
        {"name": "list_rmat15", "graph": "rmat", "scale": 15, "patterns": "ffl", "unreduced": True, "call": "list"},
        # a 5-vertex pattern on every root: leaf group of two, level reuse
        {"name": "tt4p_rmat18", "graph": "rmat", "scale": 18, "order": "ranked", "patterns": "tt4p", "call": "run"},
        # a 5-cycle with a chord on a share of the roots of a larger graph
        {"name": "c5chord_rmat20", "graph": "rmat", "scale": 20, "order": "ranked", "patterns": "c5chord",
         "share": 8, "call": "run"},
        # a burst of mixed 3-7-vertex requests through the server
        {"name": "serve_rmat19", "graph": "rmat", "scale": 19, "patterns": "serve:48", "call": "serve"},
        # the batch workload: many stored patterns of 3-6 vertices in one launch
        # on the benchmark's graph size, with its launch options
        {"name": "batch96_rmat22", "graph": "rmat", "scale": 22, "order": "ranked", "patterns": "pool:24",
         "rows_gib": 32, "tuned": True, "call": "replay"},
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))

    def some(names, most):
        return ",".join(rng.sample(names, rng.randint(1, most)))

    kind = rng.choice(["uniform", "uniform", "anchored", "subset", "motifs", "motifs", "list", "tt4p", "c5chord",
                       "serve", "batch", "batch"])
    if kind == "uniform":
        n = log(500, 40000)
        return {"graph": "uniform", "n": n, "m": n * log(4, 20) + rng.randint(0, 7),
                "patterns": some(["ffl", "c3", "bifan", "c4", "tt4p", "c5chord", "mixed_star", "outstar3", "path3"], 3),
                "unreduced": rng.random() < 0.3, "call": rng.choice(["count", "run", "replay"])}
    scale = rng.randint(12, 16)
    n = (1 << scale) - rng.randint(0, 1 << (scale - 2))
    c = {"graph": "rmat", "scale": scale, "n": n}
    if kind == "anchored":
        scale = rng.randint(14, 20)
        return {"graph": "rmat", "scale": scale, "patterns": rng.choice(["ffl", "c3", "bifan"]),
                "vertex": rng.randint(0, 2), "nodes": rng.randint(1, 8), "call": "anchored"}
    if kind == "subset":
        return {**c, "patterns": some(MOTIFS.split(","), 4), "vertex": rng.randint(0, 2),
                "percent": rng.randint(2, 60), "call": "subset"}
    if kind == "motifs":
        if rng.random() < 0.5:
            side = lambda: rng.choice(["", ":above", ":below"])  # noqa: E731
            return {**c, "order": rng.choice(["degree", "generated"]),
                    "patterns": ",".join(p + side() for p in rng.sample(MOTIFS.split(","), rng.randint(1, 4))),
                    "call": rng.choice(["count", "run", "replay"])}
        return {**c, "patterns": some(MOTIFS.split(","), 4), "unreduced": rng.random() < 0.5,
                "call": rng.choice(["count", "run", "replay"])}
    if kind == "list":
        scale = rng.randint(10, 15)
        return {"graph": "rmat", "scale": scale, "n": (1 << scale) - rng.randint(0, 1 << (scale - 2)),
                "patterns": rng.choice(["ffl", "c3"]), "unreduced": rng.random() < 0.5, "call": "list"}
    if kind == "tt4p":
        scale = rng.randint(14, 18)
        return {"graph": "rmat", "scale": scale, "order": rng.choice(["ranked", "generated"]),
                "n": (1 << scale) - rng.randint(0, 1 << (scale - 2)),
                "patterns": rng.choice(["tt4p", "tt4p_out", "tt4p_t3"]), "call": rng.choice(["count", "run"])}
    if kind == "c5chord":
        return {"graph": "rmat", "scale": rng.randint(15, 20), "order": "ranked", "patterns": "c5chord",
                "share": rng.randint(8, 10), "call": "run"}
    if kind == "serve":
        return {"graph": "rmat", "scale": rng.randint(16, 20), "patterns": "serve:%d" % log(8, 48), "call": "serve"}
    return {"graph": "rmat", "scale": rng.randint(17, 22), "order": rng.choice(["ranked", "generated"]),
            "patterns": "pool:%d" % log(2, 20), "rows_gib": rng.choice([0, 8, 16, 32]),
            "tuned": rng.random() < 0.5, "call": rng.choice(["count", "run", "replay"])}


def _arcs(case, seed):
    """Distinct arcs u * 2**32 + v (u != v), sorted, on the GPU, and the node count."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1000003 * seed + 17)
    if case["graph"] == "uniform":
        n, m = case["n"], case["m"]
        key = torch.empty(0, dtype=torch.int64, device="cuda")
        while key.numel() < m:
            u, v = torch.randint(0, n, (2, m + m // 4 + 64), generator=gen, device="cuda", dtype=torch.int64)
            key = torch.unique(torch.cat([key, ((u << 32) | v)[u != v]]))
        keep = torch.randperm(key.numel(), generator=gen, device="cuda")[:m]
        return torch.sort(key[keep])[0], n
    scale = case["scale"]
    n = case.get("n") or 1 << scale
    parts, total = [], 16 << scale
    for at in range(0, total, 1 << 24):
        cnt = min(1 << 24, total - at)
        u = torch.zeros(cnt, dtype=torch.int32, device="cuda")
        v = torch.zeros(cnt, dtype=torch.int32, device="cuda")
        for _ in range(scale):
            r = torch.rand(cnt, generator=gen, device="cuda")
            ub = r >= 0.76
            vb = ((r >= 0.57) & ~ub) | (r >= 0.95)
            u = u * 2 + ub
            v = v * 2 + vb
        ok = (u != v) & (u < n) & (v < n)
        parts.append(torch.unique((u[ok].long() << 32) | v[ok].long()))
    return (torch.unique(torch.cat(parts)) if len(parts) > 1 else parts[0]), n


def _graph(case, seed):
    key, n = _arcs(case, seed)
    src, dst = key >> 32, key & 0xFFFFFFFF
    if case.get("order") == "ranked":
        deg = torch.bincount(src, minlength=n) + torch.bincount(dst, minlength=n)
        new = torch.empty(n, dtype=torch.int64, device="cuda")
        new[torch.sort(deg, descending=True, stable=True)[1]] = torch.arange(n, device="cuda")
        key = torch.sort((new[src] << 32) | new[dst])[0]
        src, dst = key >> 32, key & 0xFFFFFFFF

    def off(major):
        o = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
        o[1:] = torch.cumsum(torch.bincount(major, minlength=n), 0)
        return o.to(torch.int32)

    g = xmgen.DeviceDigraph(n, off(src), dst.to(torch.int32), off(dst),
                            (torch.sort((dst << 32) | src)[0] & 0xFFFFFFFF).to(torch.int32))
    del key, src, dst
    if case.get("order") == "degree":
        return Graph(g.to_host(), order_by_degree=True)
    return Graph(g, dense_rows=case["rows_gib"] << 30 if case.get("rows_gib") else None)


def _plans(case, G):
    reduced = not case.get("unreduced")
    if case["patterns"].startswith("pool:"):
        per = int(case["patterns"][5:])
        got, out = {}, []
        for p, s in zip(workloads.batch_patterns(), workloads.batch_shares()):
            got[p.k] = got.get(p.k, 0) + 1
            if got[p.k] <= per:
                out.append(Plan(p, symmetry="above", root_share=s))
        return out
    out = []
    for name in case["patterns"].split(","):
        name, _, side = name.partition(":")
        out.append(Plan(xmgen.named(name), reduced=reduced, graph=G, symmetry=side or False,
                        root_share=case.get("share") or 0,
                        root_vertex=case["vertex"] if case["call"] == "subset" else None))
    return out


def prepare(case, seed):
    G = _graph(case, seed)
    rng = np.random.default_rng(seed)
    call = case["call"]
    s = {"call": call, "graph": G}
    if call == "serve":
        pool = workloads.serve_pool()
        pick = np.random.default_rng(len(pool)).permutation(len(pool))[: int(case["patterns"][6:])]
        s["requests"] = [pool[i] for i in pick]
        s["backend"] = GpuBackend({0: G})
        for p, share in s["requests"]:
            s["backend"].plan(0, p, share=share)
        return s
    if call == "anchored":
        # one node with long lists and nodes drawn from the rest of the arcs' ends
        ends = G.tensors[1].cpu().numpy()
        s["nodes"] = np.concatenate([[np.bincount(ends).argmax()], rng.choice(ends, case["nodes"] - 1)]).astype(np.uint32)
        s["pattern"], s["vertex"] = xmgen.named(case["patterns"]), case["vertex"]
        return s
    plans = s["plans"] = _plans(case, G)
    opts = {}
    if case.get("tuned"):
        opts = {"split_work": 16384, "split": 512, "chunk": 64}
    s["opts"] = opts
    if call == "subset":
        opts["roots"] = np.sort(rng.permutation(G.n)[: max(1, G.n * case["percent"] // 100)]).astype(np.uint32)
    if call == "list":
        opts["list_cap"] = 512 * G.n  # room for every row: triangles stay below it at these scales
    if call != "count":
        s["counter"] = Counter(G, plans, **opts)
        if call == "replay":
            s["stream"] = torch.cuda.Stream()
            s["counter"].capture(s["stream"])
    return s


def _split(values):
    """128-bit counts as pairs of whole numbers below 2**62."""
    return [[v & ((1 << 62) - 1), v >> 62] for v in values]


def run(s):
    call = s["call"]
    if call == "count":
        return _split(count(s["graph"], s["plans"], **s["opts"]))
    if call == "anchored":
        return _split(count_anchored(s["graph"], s["pattern"], s["vertex"], s["nodes"]))
    if call == "serve":
        srv = Server(s["backend"], 64 << 30, slots=4, max_batch=16)
        futs = [srv.submit(0, p, share=share) for p, share in s["requests"]]
        got = [f.result() for f in futs]
        srv.close()
        return np.array([_split([c])[0] + [status] for c, status in got], dtype=np.int64)
    c = s["counter"]
    c.run(s.get("stream"))
    if "stream" in s:
        torch.cuda.current_stream().wait_stream(s["stream"])
    if call == "list":
        # rows come in no particular order: one 64-bit key a row, sorted
        r = c.list.view(-1, 3).long()
        key = (r[:, 0] * s["graph"].n + r[:, 1]) * s["graph"].n + r[:, 2]
        key[torch.arange(key.numel(), device=key.device) >= c.list_count] = -1  # rows not written
        return c.counts, c.list_count, torch.sort(key)[0]
    return c.counts, c.status


def work(case):
    """The graph's two CSRs read once and the answers written."""
    if case["graph"] == "uniform":
        n, m = case["n"], case["m"]
    else:
        n = case.get("n") or 1 << case["scale"]
        m = int(0.95 * 16 * n)
    b = 8 * (n + 1) + 8 * m
    if case["call"] == "list":
        b += 4 * 3 * m
    return {"bytes": b, "flops": 0}


def exact(case, seed):
    """Counts of the motifs from adjacency-matrix identities, where the matrix is small."""
    names = case["patterns"].split(",")
    n = case.get("n") or 1 << case.get("scale", 30)
    if n > 4096 or case["call"] not in ("count", "run", "replay") or any(p.split(":")[0] not in MOTIFS.split(",") for p in names):
        return None
    key, n = _arcs(case, seed)
    A = torch.zeros(n, n, dtype=torch.float64, device="cuda")
    A[key >> 32, key & 0xFFFFFFFF] = 1.0
    A2 = A @ A
    M = A.T @ A
    M.fill_diagonal_(0.0)
    r = (A * A.T).sum(1)
    of = {"ffl": (A2 * A).sum(), "c3": (A2 * A.T).sum(), "bifan": (M * (M - 1)).sum(),
          "c4": (A2 * A2.T).sum() - 2 * (r * r).sum() + r.sum()}
    got = [int(of[p.split(":")[0]]) for p in names]
    if case["call"] == "count":
        return _split(got)
    lohi = torch.tensor([x for v in got for x in (v, 0)], dtype=torch.int64)
    return lohi, torch.zeros(len(got), dtype=torch.int32)
