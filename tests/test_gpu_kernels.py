"""Parity with the oracle at the edges of single kernels: the sizes and shapes
where a kernel's dispatch, tile or buffer ends."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

KEYS = ("count", "nodes", "children", "dead_ends", "hash_xor", "hash_sum", "omega", "hist")


@pytest.fixture(autouse=True)
def _opts(mce):
    mce.reset_options(watchdog_ms=20000)
    yield
    mce.reset_options(watchdog_ms=20000)


def same(a, b):
    for k in KEYS:
        assert a[k] == b[k], "%s: %r != %r" % (k, a[k], b[k])


def _hub(n, p, seed, deg):
    """G(n, p) with vertex n // 2 joined to exactly its first deg other vertices."""
    adj = synth.unpack_rows(synth.gnp(n, p, seed))
    v = n // 2
    adj[v, :] = adj[:, v] = False
    others = [u for u in range(n) if u != v][:deg]
    adj[v, others] = adj[others, v] = True
    return synth.pack_rows(adj)


def _cliques(n, k):
    """Disjoint cliques of k vertices (the last one of what is left)."""
    g = np.arange(n) // k
    adj = g[:, None] == g[None, :]
    np.fill_diagonal(adj, False)
    return synth.pack_rows(adj)


def _wide(rows, words):
    """The same rows with more words each."""
    out = np.zeros((rows.shape[0], words), dtype=np.uint64)
    out[:, :rows.shape[1]] = rows
    return out


@pytest.mark.parametrize("name,rows", [
    # rows too large for LDS start near 1130 vertices, or earlier when given wide
    ("n1000 wide", lambda: _wide(synth.gnp(1000, 0.02, 1), 40)),
    ("n60 wide", lambda: _wide(synth.gnp(60, 0.3, 2), 400)),
    ("n1153", lambda: synth.gnp(1153, 0.02, 3)),
    ("n2048 deg128", lambda: _hub(2048, 0.01, 4, 128)),
    ("n2048 deg129", lambda: _hub(2048, 0.01, 5, 129)),
    ("n2049", lambda: synth.gnp(2049, 0.01, 6)),
    ("n4096 deg128", lambda: _hub(4096, 0.004, 7, 128)),
    ("n4096 deg129", lambda: _hub(4096, 0.004, 8, 129)),
    ("n1500 dense", lambda: synth.gnp(1500, 0.1, 9)),
    # one pick a chunk: the list kernel leaves the graph to the other one
    ("n4096 cliques", lambda: _cliques(4096, 128)),
    ("n1300 cliques", lambda: _cliques(1300, 129)),
    ("n3000 empty", lambda: synth.empty(3000)),
    ("n2500 path", lambda: synth.path(2500)),
])
def test_order_above_lds(mce, orc, name, rows):
    import torch
    rows = rows()
    want = list(orc.order(rows))
    for r in (rows, torch.from_numpy(rows.view(np.int64)).cuda()):
        g = mce.Graph(r)
        try:
            assert list(g.order()) == want, name
        finally:
            g.release()
    if rows.shape[0] <= 2048:
        same(mce.count_noalloc(torch.from_numpy(rows.view(np.int64)).cuda()), orc.greedy(rows, threads=8))


def test_order_above_lds_batch(mce, orc):
    # lists, rows and the empty graph side by side
    graphs = [synth.gnp(1800, 0.01, 1), synth.empty(0), synth.gnp(1400, 0.15, 2), _cliques(1700, 100), synth.gnp(30, 0.5, 3)]
    b = mce.Graph(batch=graphs)
    try:
        for i, rows in enumerate(graphs):
            assert list(b.order(i)) == list(orc.order(rows)), i
    finally:
        b.release()
