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
    # largest degrees, one pick a degree, one degree for all
    ("n2049 dense", lambda: synth.gnp(2049, 0.1, 10)),
    ("n4096 dense", lambda: synth.gnp(4096, 0.5, 11)),
    ("n4095 complete", lambda: synth.complete(4095)),
    ("n4000 star", lambda: synth.star(4000)),
    ("n3000 halves", lambda: synth.complete_multipartite([1500, 1500])),
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


@pytest.mark.parametrize("small,large", [(1, 1), (6, 1), (7, 1), (8, 1), (40, 2), (0, 3)])
def test_order_mixed_batch(mce, orc, small, large):
    # a few graphs above LDS among smaller ones: ordered on lists while they
    # are at least an eighth of the batch; the small ones (at most 1024
    # vertices) never are
    sizes = [17, 300, 1024, 0, 1025, 64, 2]
    graphs = [synth.gnp(sizes[i % 7], 0.05, i) if sizes[i % 7] else synth.empty(0) for i in range(small)]
    graphs += [synth.gnp(1800 + i, 0.01, i) for i in range(large)]
    b = mce.Graph(batch=graphs)
    try:
        for i, rows in enumerate(graphs):
            assert list(b.order(i)) == list(orc.order(rows)), i
    finally:
        b.release()


def _join(a, b):
    """Every vertex of a adjacent to every vertex of b."""
    x, y = synth.unpack_rows(a), synth.unpack_rows(b)
    n, m = x.shape[0], y.shape[0]
    adj = np.ones((n + m, n + m), dtype=bool)
    adj[:n, :n] = x
    adj[n:, n:] = y
    return synth.pack_rows(adj)


def _pairs(k):
    """Complement of k disjoint edges: 2^k maximal cliques, k levels deep."""
    return synth.complete_multipartite([2] * k)


def _stairs(k):
    """A clique a_0 .. a_(k-1) and b_i joined to the a_j, j < i: k + 1 levels
    deep, with one candidate left at each."""
    a = np.zeros((2 * k, 2 * k), dtype=bool)
    a[:k, :k] = ~np.eye(k, dtype=bool)
    for i in range(k):
        a[k + i, :i] = a[:i, k + i] = True
    return synth.pack_rows(a)


# The lane search takes nodes of at most 121 vertices (two words a lane up to
# 57, three up to 89), 128 with the clique so far; its lanes keep 3 to 6 frames
# in LDS and 16 more in HBM at first.
LANE_GRAPHS = [
    ("n57", lambda: synth.gnp(57, 0.7, 1)),
    ("n58", lambda: synth.gnp(58, 0.7, 2)),
    ("n89", lambda: synth.gnp(89, 0.7, 13)),
    ("n90", lambda: synth.gnp(90, 0.7, 14)),
    ("n121", lambda: synth.gnp(121, 0.55, 3)),
    ("n122", lambda: synth.gnp(122, 0.55, 4)),
    ("degrees near 121", lambda: synth.gnp(300, 0.4, 5)),
    # universal vertices: a clique of 7 and nodes of 121, one of 8, one of 90
    ("7 + 121", lambda: _join(synth.complete(7), synth.gnp(121, 0.4, 6))),
    ("8 + 121", lambda: _join(synth.complete(8), synth.gnp(121, 0.4, 7))),
    ("90 + 60", lambda: _join(synth.complete(90), synth.gnp(60, 0.5, 8))),
    # frames past the LDS ring, and past the first levels in HBM (a second launch)
    ("pairs 16", lambda: _pairs(16)),
    ("stairs 27", lambda: _stairs(27)),
    ("stairs 43", lambda: _stairs(43)),
    ("stairs 60", lambda: _stairs(60)),
    ("hub + 3 x pairs 14", lambda: _join(synth.complete(1), synth.disjoint_union(*[_pairs(14)] * 3))),
    ("K121", lambda: synth.complete(121)),
    ("moon moser 11", lambda: synth.moon_moser(11)),
    ("n2016", lambda: synth.gnp(2016, 0.05, 9)),
    # more pieces of root units than candidates
    ("n90 dense", lambda: synth.gnp(90, 0.8, 10)),
]


@pytest.mark.parametrize("name,rows", LANE_GRAPHS)
def test_lane_search(mce, orc, name, rows):
    import torch
    rows = rows()
    ref = orc.greedy(rows, threads=8)
    g = mce.Graph(rows)
    try:
        same(g.count(), ref)
        # another schedule: few wavefronts, a look after every child
        mce.reset_options(watchdog_ms=20000, blocks=3, waves_per_block=3, check_interval=1, split_threshold=1)
        same(g.count(), ref)
        mce.reset_options(watchdog_ms=20000)
        nb = g.root_branches()
        parts = [g.count_range(a, b) for a, b in ((0, nb // 3), (nb // 3, nb))]
        assert sum(p["count"] for p in parts) == ref["count"] and sum(p["nodes"] for p in parts) == ref["nodes"]
        assert parts[0]["hash_xor"] ^ parts[1]["hash_xor"] == ref["hash_xor"]
    finally:
        g.release()
    same(mce.count_noalloc(torch.from_numpy(rows.view(np.int64)).cuda()), ref)


@pytest.mark.parametrize("name,rows,lanes", [
    # the lanes' levels run out (one wavefront, all of its lanes busy on the
    # pairs while one goes down the stairs); the loops'
    ("lanes", lambda: _join(synth.complete(1), synth.disjoint_union(_stairs(26), _pairs(16), _pairs(16))), True),
    ("loop", lambda: _stairs(200), False),
])
def test_stack_reruns(mce, orc, name, rows, lanes):
    if lanes:
        mce.reset_options(watchdog_ms=20000, blocks=1, waves_per_block=1)
    rows = rows()
    ref = orc.greedy(rows, threads=8)
    b = mce.Graph(batch=[rows, synth.complete(2)])
    try:
        for attempts in (2, 1):
            same(b.count()[0], ref)
            # what the handle learned holds for its next solve
            assert mce.last_stats()["attempts"] == attempts
    finally:
        b.release()


@pytest.mark.parametrize("rule", ("tomita_bb", "greedy_tx"))
@pytest.mark.parametrize("rows", [lambda: synth.gnp(58, 0.7, 2), lambda: synth.gnp(260, 0.4, 3), lambda: _pairs(12)])
def test_lane_search_rules(mce, orc, rows, rule):
    rows = rows()
    mce.set_option("pivot", mce.PIVOT_RULES[rule])
    g = mce.Graph(rows)
    try:
        same(g.count(), orc.solve_rule(rows, rule))
    finally:
        g.release()


def test_lane_search_lists(mce, orc):
    # the cliques themselves: listed by lanes, of a whole graph and of local graphs
    for rows in (synth.gnp(130, 0.5, 1), synth.gnp(4200, 0.02, 2)):
        ref, want = orc.greedy_list(rows)
        g = mce.Graph(rows)
        try:
            res, verts, offs = g.enumerate()
            same(res, ref)
            assert sorted(mce.cliques_from_output(verts, offs, res["count"])) == sorted(want)
        finally:
            g.release()


@pytest.mark.parametrize("rule", ("tomita_bb", "greedy_tx"))
@pytest.mark.parametrize("n,p,seed", [(130, 0.5, 1), (4200, 0.02, 2)])
def test_lane_search_rules_list(mce, orc, n, p, seed, rule):
    # lanes under the other rules: counted and listed, of a whole graph and of
    # local graphs (the cliques themselves are the same under every rule)
    rows = synth.gnp(n, p, seed)
    ref = orc.solve_rule(rows, rule)
    _, want = orc.greedy_list(rows)
    mce.set_option("pivot", mce.PIVOT_RULES[rule])
    g = mce.Graph(rows)
    try:
        same(g.count(), ref)
        res, verts, offs = g.enumerate()
        same(res, ref)
        assert sorted(mce.cliques_from_output(verts, offs, res["count"])) == sorted(want)
    finally:
        g.release()


@pytest.mark.parametrize("n,p", [(90, 0.8), (250, 0.5), (1000, 0.2), (1130, 0.2), (2016, 0.1)])
def test_noalloc_takes_one_launch(mce, orc, n, p):
    # (every wavefront has stacks in the fixed area: a search that runs out of
    # them runs again with fewer)
    import torch
    rows = synth.gnp(n, p, 1)
    same(mce.count_noalloc(torch.from_numpy(rows.view(np.int64)).cuda()), orc.greedy(rows, threads=8))
    assert mce.last_stats()["attempts"] == 1


@pytest.mark.parametrize("cap", (0, 16))
def test_batch_pieces(mce, orc, cap):
    # graphs of a batch whose root units are cut into pieces beside graphs of
    # one unit (cap = 16: no room for pieces)
    if cap:
        mce.set_option("queue_cap", cap)
    graphs = [synth.gnp(64, 0.85, 1), synth.empty(0), synth.gnp(40, 0.5, 2), synth.gnp(90, 0.75, 3),
              synth.complete(5), synth.moon_moser(10), synth.gnp(300, 0.2, 4)]
    b = mce.Graph(batch=graphs)
    try:
        for _ in range(3):
            for got, rows in zip(b.count(), graphs):
                same(got, orc.greedy(rows, threads=8))
    finally:
        b.release()


# Chains of nodes of one candidate above a node that branches: as long as every
# piece of a root unit goes down, one less and one more (64, 8 under the other
# rules), much longer, and a chain between two cuts.
@pytest.mark.parametrize("rule", ("greedy_bb", "tomita_bb", "greedy_tx"))
@pytest.mark.parametrize("name,rows", [(str(k), lambda k=k: _join(synth.complete(k), synth.gnp(70, 0.55, k)))
                                       for k in (7, 8, 9, 63, 64, 65, 300)] + [
    ("K700", lambda: synth.complete(700)),
    ("cut, chain, cut", lambda: _join(synth.gnp(30, 0.5, 1), _join(synth.complete(80), synth.gnp(30, 0.6, 2)))),
    ("two chains", lambda: _join(synth.complete(1), synth.disjoint_union(synth.complete(100), synth.complete(90)))),
])
def test_piece_chains(mce, orc, name, rows, rule):
    rows = rows()
    mce.set_option("pivot", mce.PIVOT_RULES.get(rule, 0))
    ref = orc.greedy(rows, threads=8) if rule == "greedy_bb" else orc.solve_rule(rows, rule)
    for graphs in (None, [rows, synth.gnp(40, 0.5, 1)]):
        g = mce.Graph(rows) if graphs is None else mce.Graph(batch=graphs)
        try:
            got = g.count()
            same(got if graphs is None else got[0], ref)
        finally:
            g.release()


def test_piece_chain_stops_when_cancelled(mce):
    # the chain of K_2016 under TomitaBB is a scan of up to 2016 vertices a node,
    # followed by one wavefront
    import time
    mce.set_option("pivot", mce.PIVOT_RULES["tomita_bb"])
    g = mce.Graph(synth.complete(2016))
    try:
        t = mce.submit(g)
        time.sleep(0.05)
        assert mce.cancel(t) == mce.OK
        t0 = time.monotonic()
        rc, _ = mce.poll(t, 2016)
        # (2016 nodes of some 1 ms, looked at every eighth)
        assert rc == mce.E_CANCELLED and time.monotonic() - t0 < 0.5
    finally:
        mce.set_option("pivot", 0)
        g.release()


@pytest.mark.parametrize("cap", (32, 64, 4096))
def test_batch_pieces_refused(mce, orc, cap):
    # twelve graphs of one root unit that each want more pieces than a share of
    # the spare half of the pool (16, 32 or 2048 slots): the first to ask are
    # granted theirs, the others are searched in one piece
    mce.set_option("queue_cap", cap)
    graphs = [synth.complete(96), _join(synth.complete(1), synth.gnp(64, 0.85, 1))] * 6
    want = [orc.greedy(rows, threads=8) for rows in graphs[:2]]
    b = mce.Graph(batch=graphs)
    try:
        for _ in range(3):
            for i, got in enumerate(b.count()):
                same(got, want[i % 2])
    finally:
        b.release()


def test_handles_share_stack_memory(mce, orc):
    # a handle that has been counted keeps no stacks in device memory (some
    # 200 MB a solve): many may be alive at once
    import torch
    rows = synth.gnp(100, 0.6, 1)
    ref = orc.greedy(rows)
    handles = []
    try:
        for i in range(48):
            handles.append(mce.Graph(rows))
            same(handles[-1].count(), ref)
            if i == 7:
                free = torch.cuda.mem_get_info()[0]
        assert free - torch.cuda.mem_get_info()[0] < 40 * (16 << 20)
        same(handles[0].count(), ref)
    finally:
        for g in handles:
            g.release()


def test_captured_batches_share_stack_memory(mce, orc):
    # a batch's count is captured and replayed: with the blocks of its capture,
    # or captured again when another handle has them
    import torch
    sets = [[synth.gnp(100, 0.6, i), synth.gnp(60, 0.5, i)] for i in range(3)]
    want = [[orc.greedy(rows) for rows in graphs] for graphs in sets]
    handles = []
    try:
        for i in range(30):
            handles.append(mce.Graph(batch=sets[i % 3]))
            if i == 3:
                free = torch.cuda.mem_get_info()[0]
            for k in {0, i // 2, i}:  # replays between the others' captures
                for got, ref in zip(handles[k].count(), want[k % 3]):
                    same(got, ref)
        assert free - torch.cuda.mem_get_info()[0] < 30 * (4 << 20)
        # larger stacks for another handle's solve, then replays
        other = mce.Graph(synth.gnp(1500, 0.05, 1))
        handles.append(other)
        for k in (0, 1, 2, 0, 1, 2):
            other.count()
            for got, ref in zip(handles[k].count(), want[k]):
                same(got, ref)
    finally:
        for g in handles:
            g.release()


@pytest.mark.parametrize("n,p", [(100, 0.6), (200, 0.5), (1000, 0.1), (2016, 0.03)])
def test_tuned_schedule_as_options(mce, orc, n, p):
    # the schedule that autotune reports, set option by option, is the search
    # it timed: the same launch and the same LDS
    rows = synth.gnp(n, p, 1)
    ref = orc.greedy(rows, threads=8)
    shape = ("waves_per_block", "blocks", "lds_depth", "lds_bytes_per_block")
    g = mce.Graph(rows)
    try:
        for trials in (1, 6):
            t = g.autotune(max_trials=trials)
            same(g.count(), ref)
            tuned = mce.last_stats()
            for k in ("waves_per_block", "blocks", "lds_depth", "split_threshold", "check_interval"):
                mce.set_option(k, t[k])
            h = mce.Graph(rows)
            try:
                same(h.count(), ref)
                st = mce.last_stats()
                assert [st[k] for k in shape] == [tuned[k] for k in shape]
            finally:
                h.release()
            mce.reset_options(watchdog_ms=20000)
    finally:
        g.release()


@pytest.mark.parametrize("n,p,per_cu", [(4200, 0.02, 4), (4200, 0.04, 4), (4200, 0.07, 5), (8200, 0.018, 5)])
def test_local_graph_workgroups(mce, orc, n, p, per_cu):
    # largest local graphs of about 120, 220, 365 and 195 vertices: five
    # workgroups a CU beyond 256 or with three local graphs a wavefront
    import torch
    rows = synth.gnp(n, p, 1)
    g = mce.Graph(rows)
    try:
        got = g.count()
        st = mce.last_stats()
        assert st["local_graphs"] > 0
        assert st["blocks"] == per_cu * torch.cuda.get_device_properties(0).multi_processor_count
        mce.set_option("local_graphs", 0)
        h = mce.Graph(rows)
        try:
            same(got, h.count())
        finally:
            h.release()
    finally:
        g.release()


@pytest.mark.parametrize("n,p,depth", [(2016, 0.03, 12), (2016, 0.03, 5), (1000, 0.05, 11), (300, 0.3, 3)])
def test_window_without_lanes(mce, orc, n, p, depth):
    # a window asked for that is not the one beside the lanes' stacks: the
    # search without lanes, in its own workgroups of eight wavefronts, has it
    mce.set_option("lds_depth", depth)
    rows = synth.gnp(n, p, 1)
    g = mce.Graph(rows)
    try:
        same(g.count(), orc.greedy(rows, threads=8))
        st = mce.last_stats()
        assert (st["lds_depth"], st["waves_per_block"]) == (depth, 8)
    finally:
        g.release()


def test_many_workgroups(mce, orc):
    # as many workgroups as an option takes with a wavefront each: stacks of the
    # lanes for all of them would not fit in device memory
    rows = synth.gnp(300, 0.3, 1)
    ref = orc.greedy(rows, threads=8)
    for blocks, wpb in ((1 << 16, 1), ((1 << 16) + 1, 1), (1 << 19, 8)):
        mce.reset_options(watchdog_ms=20000, blocks=blocks, waves_per_block=wpb)
        g = mce.Graph(rows)
        try:
            same(g.count(), ref)
        finally:
            g.release()


@pytest.mark.parametrize("n,p", [(120, 0.6), (400, 0.3)])
def test_split_threshold_binds_lanes(mce, orc, n, p):
    # nothing is handed over from nodes of fewer vertices than the threshold
    rows = synth.gnp(n, p, 1)
    ref = orc.greedy(rows, threads=8)
    g = mce.Graph(rows)
    try:
        same(g.count(), ref)
        assert mce.last_stats()["donations"] > 0
        mce.set_option("split_threshold", 1 << 20)
        same(g.count(), ref)
        assert mce.last_stats()["donations"] == 0
    finally:
        g.release()


@pytest.mark.parametrize("n,p,waves,per_cu", [(1600, 0.05, 8, 1), (1600, 0.08, 8, 2), (1600, 0.15, 11, 1), (1020, 0.102, 8, 2),
                                              (1020, 0.08, 8, 1), (1020, 0.13, 12, 1), (300, 0.1, 8, 1), (300, 0.4, 12, 1)])
def test_lanes_by_density(mce, orc, n, p, waves, per_cu):
    # without lanes (two workgroups a CU) where neighbourhoods are too large for
    # them and common ones too small, twelve wavefronts or as many as fit where
    # there is much to do: rows in host memory, in device memory, wider ones,
    # and the entry that allocates nothing
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows = synth.gnp(n, p, 1)
    ref = orc.greedy(rows, threads=8)
    wide = np.zeros((n, rows.shape[1] + 3), dtype=np.uint64)
    wide[:, :rows.shape[1]] = rows
    dev = torch.from_numpy(wide.view(np.int64)).cuda()
    for r in (rows, wide, dev):
        g = mce.Graph(r)
        try:
            same(g.count(), ref)
            st = mce.last_stats()
            assert (st["waves_per_block"], st["blocks"]) == (waves, per_cu * cus)
        finally:
            g.release()
    same(mce.count_noalloc(dev), ref)
    st = mce.last_stats()
    assert (st["waves_per_block"], st["blocks"]) == (waves, per_cu * cus)


@pytest.mark.parametrize("n,p", [(200, 0.4), (2100, 0.03), (4300, 0.01), (8200, 0.004)])
@pytest.mark.parametrize("cap", (0, 2, 64))
def test_subproblem_units(mce, orc, n, p, cap):
    # a node's candidates in as many units as the pool holds, one to eight words
    # a lane: the root, a node with vertices in X, one with nothing to branch on
    if cap:
        mce.set_option("queue_cap", cap)
    rows = synth.gnp(n, p, 1)
    g = mce.Graph(rows)
    try:
        whole = g.count()
        same(g.count_subproblem([], range(n), []), whole)
        od = [int(v) for v in g.order()]
        adj = synth.unpack_rows(rows)[np.ix_(od, od)]
        v = max(range(n // 4), key=lambda u: int(adj[u, u:].sum()))
        nb = [int(u) for u in np.nonzero(adj[v])[0]]
        P, X = [u for u in nb if u > v], [u for u in nb if u < v]
        got = g.count_subproblem([v], P, X)
        ref = orc.subproblem(synth.pack_rows(adj), [v], P, X, ids=od)
        for k in KEYS:
            assert got[k] == ref[k], k
        # the only candidate adjacent to a vertex of X: no child, one node
        u = nb[0]
        got = g.count_subproblem([], [u], [v])
        assert (got["nodes"], got["children"], got["count"]) == (1, 0, 0)
    finally:
        g.release()


def test_batch_of_sparse_graphs_takes_few_units(mce, orc):
    # (some 25,000 root children in all: a unit for each would keep the
    # fetchers of the workgroups busy longer than the search itself)
    graphs = [synth.gnp(100, 0.1, i) for i in range(8)]
    want = [orc.greedy(rows) for rows in graphs]
    b = mce.Graph(batch=graphs * 40)
    try:
        for i, got in enumerate(b.count()):
            same(got, want[i % 8])
        assert mce.last_stats()["units"] < 10000
    finally:
        b.release()


def test_batch_lanes_by_density(mce, orc):
    # half of a batch's graphs of the kind that lanes do not suit, or less
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    large, small = synth.gnp(1200, 0.095, 1), synth.gnp(100, 0.3, 2)
    want = [orc.greedy(rows, threads=8) for rows in (large, small)]
    for graphs, per_cu in (([large, small], 2), ([large, small, small], 1)):
        b = mce.Graph(batch=graphs)
        try:
            for got, rows in zip(b.count(), graphs):
                same(got, want[0 if rows is large else 1])
            assert mce.last_stats()["blocks"] == per_cu * cus
        finally:
            b.release()


def test_batch_units(mce, orc):
    # graphs of a batch with more root children than units: a unit covers
    # several, cut into pieces where the graph is dense; and with more graphs
    # than wavefronts, each one unit
    graphs = [synth.gnp(300, 0.05, 1), synth.gnp(90, 0.75, 2), synth.empty(50), synth.star(40), synth.gnp(500, 0.1, 3)]
    want = [orc.greedy(rows, threads=8) for rows in graphs]
    for opts in ({}, {"blocks": 2, "waves_per_block": 2}, {"blocks": 1, "waves_per_block": 1, "queue_cap": 16}):
        mce.reset_options(watchdog_ms=20000, **opts)
        for copies in (1, 9):
            b = mce.Graph(batch=graphs * copies)
            try:
                for i, got in enumerate(b.count()):
                    same(got, want[i % len(graphs)])
            finally:
                b.release()


def test_served_jobs_keep_their_wavefronts(mce, orc):
    # a sparse graph's count takes workgroups of eight wavefronts; served, its
    # share is a number of workgroups, of twelve
    rows = synth.gnp(300, 0.2, 1)
    ref = orc.greedy(rows)
    g = mce.Graph(rows)
    try:
        same(g.count(), ref)
        assert mce.last_stats()["waves_per_block"] == 8
        for t in [mce.submit(g) for _ in range(3)]:
            rc, got = mce.poll(t, 300)
            assert rc == mce.OK
            same(got, ref)
    finally:
        g.release()
