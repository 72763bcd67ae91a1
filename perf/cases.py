"""Workloads of the maximal clique library, as a program that uses it runs them.

``listed()`` gives the standing cases, ``draw(rng)`` one more of the same
ranges.  A case names how the library is called ("how") and the random graph
G(n, p) it is called on:

  job        rows in device memory -> Graph, count, release
  host       the same from a numpy array in host memory
  noalloc    count_noalloc on rows in device memory
  count      count on a handle that the program keeps
  enumerate  enumerate on a kept handle into kept device buffers
  batch      many graphs in one handle: Graph(batch=...), count, release
  serve      requests submitted as they come in, each with a graph of its own,
             then polled and released
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_1801_00202_amd import mce

MASK = (1 << 64) - 1


def listed():
    return [
        # one tiny graph: what a single call costs
        {"name": "job_n40_p05", "how": "job", "n": 40, "p": 0.5, "pivot": "greedy"},
        # a graph read from a file: rows in host memory (a row of Table 1)
        {"name": "host_n500_p02", "how": "host", "n": 500, "p": 0.2, "pivot": "greedy"},
        # the benchmark's workload and the heaviest n = 1000 row of Table 1
        {"name": "job_n1000_p03", "how": "job", "n": 1000, "p": 0.3, "pivot": "greedy"},
        # medium density, where cliques overlap most
        {"name": "job_n300_p05", "how": "job", "n": 300, "p": 0.5, "pivot": "greedy"},
        # small and dense: a deep search on few vertices
        {"name": "job_n100_p075", "how": "job", "n": 100, "p": 0.75, "pivot": "greedy"},
        # another pivot rule on a handle kept between calls
        {"name": "count_n500_p03_tomita", "how": "count", "n": 500, "p": 0.3, "pivot": "tomita_bb"},
        # a few thousand vertices (rows of two words a lane)
        {"name": "job_n3500_p001", "how": "job", "n": 3500, "p": 0.01, "pivot": "greedy"},
        # Table 1's n = 10^4 graphs, the sparsest and the densest
        {"name": "job_n10000_p0001", "how": "job", "n": 10000, "p": 0.001, "pivot": "greedy"},
        {"name": "job_n10000_p003", "how": "job", "n": 10000, "p": 0.03, "pivot": "greedy"},
        # the cliques themselves, not only their totals
        {"name": "enumerate_n600_p02", "how": "enumerate", "n": 600, "p": 0.2, "pivot": "greedy"},
        # a batch of graphs of mixed sizes
        {"name": "batch_384", "how": "batch", "graphs": 384, "n_lo": 32, "n_hi": 512, "p_lo": 0.1, "p_hi": 0.9,
         "mu_cap": 1e6, "specs": 7, "pivot": "greedy"},
        # requests of mixed sizes that come in together
        {"name": "serve_16", "how": "serve", "graphs": 16, "n_lo": 64, "n_hi": 2048, "p_lo": 0.2, "p_hi": 0.9,
         "mu_cap": 1e6, "specs": 5, "pivot": "greedy"},
    ]


def draw(rng):
    how = rng.choice(["job", "job", "job", "host", "noalloc", "count", "enumerate", "batch", "serve"])
    if how == "batch":
        return {"how": how, "graphs": rng.randint(24, 300), "n_lo": rng.randint(16, 64), "n_hi": rng.randint(128, 512),
                "p_lo": 0.1, "p_hi": 0.9, "mu_cap": 1e6, "specs": rng.randrange(1 << 20), "pivot": "greedy"}
    if how == "serve":
        return {"how": how, "graphs": rng.randint(6, 24), "n_lo": 64, "n_hi": 2048, "p_lo": 0.2, "p_hi": 0.9,
                "mu_cap": 1e6, "specs": rng.randrange(1 << 20), "pivot": "greedy"}
    pivot = rng.choice(["greedy", "tomita_bb", "greedy_tx"]) if how == "count" else "greedy"
    top = {"job": 10000, "host": 5000, "noalloc": 2048, "count": 3000, "enumerate": 3000}[how]
    cap = {"job": 1.2e7, "host": 4e6, "noalloc": 2e6, "count": 2e6, "enumerate": 1e6}[how]
    while True:
        n = round(math.exp(rng.uniform(math.log(17), math.log(top))))
        p = round(math.exp(rng.uniform(math.log(0.001), math.log(0.9))), 4)
        # neither an edgeless graph nor one of more cliques than the listed
        # ones (a denser search looks at more nodes for each clique)
        if p * n >= 4 and expected_cliques(n, p) <= (cap if p <= 0.6 else cap / 8):
            return {"how": how, "n": n, "p": p, "pivot": pivot}


def expected_cliques(n, p):
    """E[maximal cliques] of G(n, p): sum over k of C(n, k) p^C(k, 2) (1 - p^k)^(n - k)."""
    total = 0.0
    for k in range(1, n + 1):
        t = (math.lgamma(n + 1) - math.lgamma(k + 1) - math.lgamma(n - k + 1) + k * (k - 1) / 2 * math.log(p)
             + (n - k) * math.log1p(-p ** k))
        total += math.exp(t) if t > -700 else 0.0
        if k > 4 and t < -40 and p ** k * n < 1e-3:
            break
    return total


def specs(case):
    """(n, p) of each graph of a case."""
    if "graphs" not in case:
        return [(case["n"], case["p"])]
    rng, got = random.Random(case["specs"]), []
    while len(got) < case["graphs"]:
        if case["how"] == "serve":
            n = round(math.exp(rng.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]))))
        else:
            n = rng.randint(case["n_lo"], case["n_hi"])
        p = rng.uniform(case["p_lo"], case["p_hi"])
        if expected_cliques(n, p) <= case["mu_cap"]:
            got.append((n, p))
    return got


def gnp(n, p, gen, device):
    """Adjacency rows of G(n, p), int64[n, ceil(n / 64)] (bit j of row i: an edge)."""
    words = (n + 63) // 64
    a = torch.zeros(n, words * 64, dtype=torch.bool, device=device)
    a[:, :n] = torch.rand(n, n, generator=gen, device=device) < p
    a[:, :n].triu_(1)
    a[:, :n] |= a[:, :n].T.clone()
    weights = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.uint8, device=device)
    out = torch.empty(n, words * 8, dtype=torch.uint8, device=device)
    for i in range(0, n, 1024):
        out[i:i + 1024] = (a[i:i + 1024].view(-1, words * 8, 8).to(torch.uint8) * weights).sum(-1, dtype=torch.uint8)
    return out.view(torch.int64)


def inputs(case, seed):
    """The rows of the case's graphs: device tensors, or host arrays for "host" and "batch"."""
    if case["how"] in ("host", "batch"):
        rng, got = np.random.default_rng(seed), []
        for n, p in specs(case):
            words = (n + 63) // 64
            a = np.zeros((n, words * 64), dtype=bool)
            a[:, :n] = np.triu(rng.random((n, n), dtype=np.float32) < p, 1)
            a[:, :n] |= a[:, :n].T.copy()
            got.append(np.packbits(a, axis=1, bitorder="little").view(np.uint64))
        return got
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [gnp(n, p, gen, "cuda") for n, p in specs(case)]


def prepare(case, seed):
    state = {"how": case["how"], "pivot": case["pivot"], "rows": inputs(case, seed)}
    if case["how"] in ("count", "enumerate"):
        state["graph"] = mce.Graph(state["rows"][0])
    if case["how"] == "enumerate":
        # output buffers of the size a count asks for; a 64-bit key a vertex
        # (a clique's key is the sum of its vertices' keys) and a table for
        # the cliques' keys
        hist = state["graph"].count()["hist"]
        state["verts"] = torch.zeros(sum(k * c for k, c in enumerate(hist)), dtype=torch.int32, device="cuda")
        state["offsets"] = torch.zeros(2 * sum(hist), dtype=torch.int64, device="cuda")
        state["keys"] = torch.from_numpy(vertex_keys(case["n"], seed)).cuda()
        state["table"] = torch.zeros(table_size(case), dtype=torch.int64, device="cuda")
    return state


def table_size(case):
    return 4096 + 2 * int(expected_cliques(case["n"], case["p"]))


def vertex_keys(n, seed):
    return np.random.default_rng([seed, 1]).integers(-1 << 62, 1 << 62, n, dtype=np.int64)


def totals(results):
    """The totals of one or more graphs, field by field."""
    out = {k: np.array([r[k] for r in results], dtype=np.uint64)
           for k in ("count", "nodes", "children", "dead_ends", "hash_xor", "hash_sum", "omega")}
    # the binding drops the zeros at the end of a histogram: 512 sizes are kept
    out["hist"] = np.zeros((len(results), 512), dtype=np.uint64)
    for row, r in zip(out["hist"], results):
        row[:len(r["hist"])] = r["hist"]
    return out


def whole_job(rows):
    g = mce.Graph(rows)
    res = g.count()
    g.release()
    return res


def run(state):
    how, rows = state["how"], state["rows"]
    if how in ("job", "host"):
        return totals([whole_job(rows[0])])
    if how == "noalloc":
        return totals([mce.count_noalloc(rows[0])])
    if how == "count":
        if state["pivot"] == "greedy":
            return totals([state["graph"].count()])
        mce.set_option("pivot", mce.PIVOT_RULES[state["pivot"]])
        try:
            return totals([state["graph"].count()])
        finally:
            mce.set_option("pivot", mce.DEFAULTS["pivot"])
    if how == "enumerate":
        # the order of the cliques is unspecified: the program keeps each
        # clique's key, sorted
        res, verts, offsets = state["graph"].enumerate(state["verts"], state["offsets"])
        ends = torch.cumsum(state["keys"][verts.long()], 0)
        ends = torch.cat([ends.new_zeros(1), ends])
        at = offsets.view(-1, 2)
        state["table"][:len(at)] = (ends[at[:, 1]] - ends[at[:, 0]]).sort().values
        return {**totals([res]), "keys": state["table"]}
    if how == "batch":
        g = mce.Graph(batch=rows)
        res = g.count()
        g.release()
        return totals(res)
    # serve
    graphs, tickets, done = [], [], []
    for r in rows:
        graphs.append(mce.Graph(r))
        tickets.append(mce.submit(graphs[-1]))
    for g, t, r in zip(graphs, tickets, rows):
        status, res = mce.poll(t, r.shape[0])
        if status != mce.OK:
            raise mce.MceError(status, "poll")
        done.append(res)
        g.release()
    return totals(done)


def work(case):
    # the rows once, the totals once; each maximal clique is at least one
    # candidate looked at: two ANDs and two tests for zero over its words
    bytes_, ops = 0.0, 0.0
    for n, p in specs(case):
        cliques = expected_cliques(n, p)
        bytes_ += n * ((n + 63) // 64) * 8 + 8 * (n + 9)
        ops += 4 * ((n + 31) // 32) * cliques
        if case["how"] == "enumerate":
            bytes_ += cliques * (8 + 16 + 4 * max(2.0, math.log(n) / -math.log(p)))
    return {"bytes": bytes_, "flops": ops}


# ---------------------------------------------------------------- oracle --


def exact(case, seed):
    """The totals by a plain search, for graphs of few cliques (Python
    integers as bitsets, the ordering and pivot of the library's method)."""
    if sum(expected_cliques(n, p) for n, p in specs(case)) > 2.5e5:
        return None
    results, lists = [], []
    for rows in inputs(case, seed):
        rows = rows.cpu().numpy().view(np.uint64) if isinstance(rows, torch.Tensor) else rows
        res, cliques = search(rows)
        results.append(res)
        lists.append(cliques)
    out = totals(results)
    if case["pivot"] != "greedy":
        out["nodes"] = out["children"] = out["dead_ends"] = None
    if case["how"] == "enumerate":
        keys = vertex_keys(case["n"], seed)
        out["keys"] = np.zeros(table_size(case), dtype=np.int64)
        out["keys"][:results[0]["count"]] = np.sort(np.concatenate([keys[c].sum(1) for c in lists[0]]))
    return out


def search(rows):
    n = rows.shape[0]
    adj = np.unpackbits(np.ascontiguousarray(rows).view(np.uint8), axis=1, bitorder="little")[:, :n].astype(bool)
    # maximum-degree-first in the remaining graph, ties to the smaller id
    degree, order = adj.sum(1).astype(np.int64), []
    for _ in range(n):
        v = int(degree.argmax())
        order.append(v)
        degree[adj[v]] -= 1
        degree[v] = -n - 1
    order = np.array(order)
    packed = np.packbits(adj[np.ix_(order, order)], axis=1, bitorder="little")
    near = [int.from_bytes(r.tobytes(), "little") for r in packed]
    found, stats = [], {"nodes": 0, "children": 0, "dead_ends": 0}

    def node(clique, P, X):
        stats["nodes"] += 1
        first = X or P
        L = P & ~near[(first & -first).bit_length() - 1]
        while L:
            bit = L & -L
            L ^= bit
            v = bit.bit_length() - 1
            stats["children"] += 1
            inner, outer = P & near[v], X & near[v]
            if inner:
                node(clique + (v,), inner, outer)
            elif outer:
                stats["dead_ends"] += 1
            else:
                found.append(clique + (v,))
            P ^= bit
            X |= bit

    node((), (1 << n) - 1, 0)
    longest = max(len(c) for c in found)
    hist = np.bincount([len(c) for c in found], minlength=longest + 1)
    lists = [np.sort(order[np.array([c for c in found if len(c) == k])], axis=1)
             for k in range(1, longest + 1) if hist[k]]
    h = np.concatenate([clique_hash(c) for c in lists])
    return {**stats, "count": len(found), "omega": longest, "hist": hist.tolist(),
            "hash_xor": int(np.bitwise_xor.reduce(h)), "hash_sum": int(h.sum(dtype=np.uint64))}, lists


def mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def clique_hash(cliques):
    """The hash of each clique of one size (rows of sorted input ids)."""
    h = mix64(np.full(len(cliques), cliques.shape[1], dtype=np.uint64))
    for i in range(cliques.shape[1]):
        h = mix64(h + np.uint64(0x9E3779B97F4A7C15) + cliques[:, i].astype(np.uint64))
    return h
