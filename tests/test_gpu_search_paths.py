"""GPU tests of the search kernels' own edges: hubs around the sizes at which the hash-set and bitmap
searches cut an entry into slices, both visited sets on the same inputs, and edge scans whose tiles end
inside a source.  Expected values come from the oracle or from plain numpy set operations."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rpq():
    import torch
    import paper_2602_20748_amd as m
    assert torch.cuda.is_available()
    m.load_library()
    return m


def hub_graph(n, hub_degrees, extra, seed):
    """Vertices 0, 1, ... are hubs of the given out-degrees over two labels; the rest is random."""
    rng = np.random.default_rng(seed)
    src, dst, lab = [], [], []
    for h, d in enumerate(hub_degrees):
        src.append(np.full(d, h))
        dst.append(rng.choice(n, size=d, replace=False))
        lab.append(rng.integers(0, 2, size=d))
    src.append(rng.integers(0, n, size=extra))
    dst.append(rng.integers(0, n, size=extra))
    lab.append(rng.integers(0, 3, size=extra))
    return (np.concatenate(src).astype(np.uint32), np.concatenate(lab).astype(np.uint8),
            np.concatenate(dst).astype(np.uint32))


@pytest.mark.parametrize("form", ["bitmap", "hash set"])
@pytest.mark.parametrize("reverse", [False, True])
def test_sparse_slices_and_visited_sets(rpq, form, reverse):
    import torch
    n = 6000
    src, lab, dst = hub_graph(n, [31, 32, 33, 255, 256, 257, 512, 513, 4000], 5000, seed=5)
    g = rpq.rpq_graph_create(src, lab, dst, n, 3, flags=rpq.RPQ_BUILD_IN_CSR, names=["a", "b", "c"])
    if reverse:
        og = oracle.OracleGraph(n, dst, lab, src, 3, ["a", "b", "c"])
    else:
        og = oracle.OracleGraph(n, src, lab, dst, 3, ["a", "b", "c"])
    # the starting workspace holds 2^16 slots: a bitmap of 9 sources is smaller, one of 400 sources is not
    sources = np.arange(9 if form == "bitmap" else 400, dtype=np.uint32)
    for rx, back in (("a.b?", "b?.a"), ("(a|b).c*", "c*.(a|b)"), ("a", "a")):
        nfa = rpq.rpq_nfa_compile(rx, g.names)
        flags = rpq.RPQ_SPARSE | (rpq.RPQ_REVERSE if reverse else 0)
        want = oracle.rpq(og, back if reverse else rx, sources=sources)
        print("case: %s reverse=%s %s" % (form, reverse, rx), flush=True)
        ws = torch.empty(rpq.rpq_eval_workspace_size(g, nfa, len(sources), flags), dtype=torch.uint8, device="cuda")
        buf = torch.zeros(max(1, want.count), dtype=torch.int64, device="cuda")
        try:
            got = rpq.rpq_eval(g, nfa, sources, flags=flags, pairs=buf, per_source=True, workspace=ws)
        except rpq.RpqError as e:
            assert e.code == rpq.RPQ_ENOMEM   # reaches more than 2^15 triples: the binding grows its own workspace
            got = rpq.rpq_eval(g, nfa, sources, flags=flags, pairs=buf, per_source=True)
        assert (got.count, got.hash) == (want.count, want.hash), rx
        assert np.array_equal(got.pairs.cpu().numpy().view(np.uint64), want.pairs), rx
        assert np.array_equal(got.per_source.cpu().numpy().view(np.uint64), want.per_source), rx
        if not reverse:
            assert got.product_edges == want.product_edges, rx
    g.close()


@pytest.mark.parametrize("rx,labels", [("a", [0]), ("a|b", [0, 1]), ("c", [2])])
@pytest.mark.parametrize("bound", [None, 8])
def test_edge_scan_tiles(rpq, rx, labels, bound):
    """One edge-scan atom: from every vertex, or from the hub of 4,000 edges alone; and backwards."""
    n = 6000
    src, lab, dst = hub_graph(n, [1, 63, 64, 65, 511, 512, 513, 1025, 4000], 3000, seed=6)
    g = rpq.rpq_graph_create(src, lab, dst, n, 3, flags=rpq.RPQ_BUILD_IN_CSR, names=["a", "b", "c"])
    keep = np.isin(lab, labels) & ((src == bound) if bound is not None else True)
    pairs = np.unique(np.stack([src[keep], dst[keep]], axis=1), axis=0)
    domain = np.arange(0, n, 3, dtype=np.uint32)
    r = rpq.crpq_eval(g, [(0, rx, 1)], 2, binding=[bound, None], tuples=True)
    want = pairs if bound is None else pairs[:, 1:]
    assert r.count == len(want) and r.atom_strategy[0] & 0xFF == 1, (r.count, len(want), r.atom_strategy)
    assert np.array_equal(r.tuples.cpu().numpy().view(np.uint32), want)
    few = rpq.crpq_eval(g, [(0, rx, 1)], 2, binding=[bound, None], domain=[None, domain], tuples=True)
    want = pairs[np.isin(pairs[:, 1], domain)][:, 0 if bound is None else 1:]
    assert np.array_equal(few.tuples.cpu().numpy().view(np.uint32), want)
    g.close()


def same_as_oracle(got, want, keys=True):
    assert (got.count, got.hash, got.product_edges) == (want.count, want.hash, want.product_edges)
    assert np.array_equal(got.per_source.cpu().numpy().view(np.uint64), want.per_source)
    if keys:
        assert np.array_equal(got.pairs.cpu().numpy().view(np.uint64), want.pairs)


def evaluate(rpq, g, nfa, sources, want, keys=True, flags=0, **opts):
    import torch
    buf = torch.zeros(max(1, want.count), dtype=torch.int64, device="cuda") if keys else None
    return rpq.rpq_eval(g, nfa, sources, flags=flags, opts=opts or None, pairs=buf, per_source=True)


@pytest.mark.parametrize("n", [70, 4096, 4097])
def test_small_graph_search(rpq, n):
    """Four states: 16,384 rows fit in LDS at 4,096 vertices and go by levels at 4,097.  Rows of 1 to 9 and of
    many edges; 31 to 33 sources a block; the empty word; bounds; in-edges; a bitmap of dead sources."""
    src, lab, dst = hub_graph(n, [1, 4, 5, 8, 9, 40, 64], 3 * n, seed=n)
    g = rpq.rpq_graph_create(src, lab, dst, n, 3, flags=rpq.RPQ_BUILD_IN_CSR, names=["a", "b", "c"])
    og = oracle.OracleGraph(n, src, lab, dst, 3, ["a", "b", "c"])
    ogt = oracle.OracleGraph(n, dst, lab, src, 3, ["a", "b", "c"])
    for rx, back in (("a.b*.c", "c.b*.a"), ("(a|b)*", "(a|b)*"), ("a?.c", "c.a?")):
        nfa = rpq.rpq_nfa_compile(rx, g.names)
        for k in (1, 31, 32, 33, 65):
            s = np.unique(np.linspace(0, n - 1, k).astype(np.uint32))
            print("case: %d vertices, %s, %d sources" % (n, rx, len(s)), flush=True)
            same_as_oracle(evaluate(rpq, g, nfa, s, want := oracle.rpq(og, rx, sources=s)), want)
        for bound in (0, 1, 2):
            want = oracle.rpq(og, rx, sources=s, max_length=bound)
            got = evaluate(rpq, g, nfa, s, want, flags=rpq.RPQ_LENGTH_BOUND, max_length=bound)
            level = evaluate(rpq, g, nfa, s, want, flags=rpq.RPQ_LENGTH_BOUND, max_length=bound, sync_every=1)
            same_as_oracle(got, want)
            assert (got.levels, got.max_depth) == (level.max_depth + 1, level.max_depth)
        want = oracle.rpq(ogt, back, sources=s)
        got = evaluate(rpq, g, nfa, s, want, flags=rpq.RPQ_REVERSE)
        assert (got.count, got.hash) == (want.count, want.hash)
        assert np.array_equal(got.pairs.cpu().numpy().view(np.uint64), want.pairs)
    g.close()


@pytest.mark.parametrize("rx", ["a.b*.c", "(a.b)*", "b?"])
@pytest.mark.parametrize("opts", [dict(sync_every=3), dict(batch_width=64, concurrency=2),
                                  dict(batch_width=128, concurrency=3, visit=1)])
def test_plain_search_of_ordered_sources(rpq, rx, opts):
    """Sources without a first edge, the empty word with and without keys, 512 and 513 sources (ordered from
    there on), several groups, both visit schemes."""
    n = 6000
    src, lab, dst = hub_graph(n, [600, 3000, 17, 16, 15], 9000, seed=9)
    g = rpq.rpq_graph_create(src, lab, dst, n, 3, names=["a", "b", "c"])
    og = oracle.OracleGraph(n, src, lab, dst, 3, ["a", "b", "c"])
    nfa = rpq.rpq_nfa_compile(rx, g.names)
    for k in (64, 65, 512, 513, 1500):
        s = np.unique(np.linspace(0, n - 1, k).astype(np.uint32))
        want = oracle.rpq(og, rx, sources=s)
        for keys in (True, False):
            print("case: %s, %d sources, %s, keys %s" % (rx, len(s), opts, keys), flush=True)
            same_as_oracle(evaluate(rpq, g, nfa, s, want, keys, **opts), want, keys)
    g.close()


@pytest.mark.parametrize("reverse", [False, True])
@pytest.mark.parametrize("rx", ["a.b", "a.b*.c", "(a|d)?.c", "d?"])
def test_rows_of_reachable_vertices(rpq, rx, reverse):
    """Bitmaps above 64 MB: rows only for the vertices that a state's labels lead to, and one a source for a
    state that nothing leads to.  The hash-set search, which has none of this, gives the expected values."""
    import torch
    n, m = 300_000, 240_000
    rng = np.random.default_rng(31)
    src, dst = rng.integers(0, n, m).astype(np.uint32), rng.integers(0, n, m).astype(np.uint32)
    lab = rng.choice(4, size=m, p=[0.3, 0.3, 0.3, 0.1]).astype(np.uint8)
    dst[lab == 3] = dst[lab == 3] % 1000
    g = rpq.rpq_graph_create(src, lab, dst, n, 4, flags=rpq.RPQ_BUILD_IN_CSR, names=["a", "b", "c", "d"])
    nfa = rpq.rpq_nfa_compile(rx, g.names)
    s = np.unique(rng.integers(0, n, 9000)).astype(np.uint32)
    flags = rpq.RPQ_REVERSE if reverse else 0
    want = rpq.rpq_eval(g, nfa, s, flags=flags | rpq.RPQ_SPARSE, pairs=True, per_source=True)
    for opts in (None, dict(batch_width=1024, concurrency=4), dict(batch_width=2048, visit=1)):
        for keys in (True, False):
            print("case: %s reverse %s %s keys %s" % (rx, reverse, opts, keys), flush=True)
            got = rpq.rpq_eval(g, nfa, s, flags=flags, opts=opts, pairs=keys or None, per_source=True)
            assert (got.count, got.hash, got.product_edges) == (want.count, want.hash, want.product_edges)
            assert torch.equal(got.per_source, want.per_source)
            assert not keys or torch.equal(got.pairs, want.pairs)
    g.close()


@pytest.mark.parametrize("leaves", [65_534, 65_536, 70_000])
@pytest.mark.parametrize("bound", [None, 2])
def test_sparse_search_hands_over(rpq, leaves, bound):
    """A star of 65,534 leaves keeps the hash-set search below 2^16 triples; larger ones are handed to the
    bit-parallel search.  Keys and tallies against the bitmap form."""
    import torch
    n = leaves + 10
    src = np.concatenate([np.zeros(leaves), np.arange(10, 110)]).astype(np.uint32)
    dst = np.concatenate([np.arange(10, 10 + leaves), np.arange(1, 101) % 9 + 1]).astype(np.uint32)
    lab = np.concatenate([np.zeros(leaves), np.ones(100)]).astype(np.uint8)
    g = rpq.rpq_graph_create(src, lab, dst, n, 2, flags=rpq.RPQ_BUILD_IN_CSR, names=["a", "b"])
    flags = rpq.RPQ_LENGTH_BOUND if bound is not None else 0
    opts = dict(max_length=bound) if bound is not None else None
    for rx, s, rev in (("a.b?", [0], 0), ("a*", [0, 3, 20], 0), ("a.b?", [1, 10, 11], rpq.RPQ_REVERSE)):
        nfa = rpq.rpq_nfa_compile(rx, g.names)
        s = np.array(s, dtype=np.uint32)
        want = rpq.rpq_eval(g, nfa, s, flags=flags | rev, opts=opts, pairs=True, per_source=True)
        got = rpq.rpq_eval(g, nfa, s, flags=flags | rev | rpq.RPQ_SPARSE, opts=opts, pairs=True,
                           per_source=True)
        print("case: %d leaves, %s, bound %s" % (leaves, rx, bound), flush=True)
        assert (got.count, got.hash, got.product_edges) == (want.count, want.hash, want.product_edges)
        assert torch.equal(got.pairs, want.pairs) and torch.equal(got.per_source, want.per_source)
    g.close()


def test_batch_segments_and_dead_sources(rpq):
    """Queries of 4,095 to 4,097 sources (a block prepares 4,096), one whose sources all lack a first edge,
    and one of only such sources whose walks of length zero count."""
    import torch
    n = 9000
    src, lab, dst = hub_graph(n, [600, 3000, 17, 16, 15], 9000, seed=10)
    keep = (src < 4500) | (lab != 2)
    src, lab, dst = src[keep], lab[keep], dst[keep]
    g = rpq.rpq_graph_create(src, lab, dst, n, 3, names=["a", "b", "c"])
    dead = np.setdiff1d(np.arange(n), src[lab == 2]).astype(np.uint32)
    some = [np.arange(k, dtype=np.uint32) * 2 % n for k in (4095, 4096, 4097)]
    queries = [(rx, np.unique(s)) for s in some for rx in ("a.b*.c", "(a.b)*")]
    queries += [("c.a", dead[:700]), ("c?", dead[:700]), ("c*.a", dead[-1:]), ("a", np.arange(1, dtype=np.uint32))]
    for width in (0, 64, 1024):
        for keys in (True, False):
            b = rpq.rpq_batch_create(g, dict(batch_width=width) if width else None)
            want = []
            for rx, s in queries:
                nfa = rpq.rpq_nfa_compile(rx, g.names)
                w = rpq.rpq_eval(g, nfa, s, opts=dict(sync_every=4), per_source=True)
                if keys:
                    w = rpq.rpq_eval(g, nfa, s, opts=dict(sync_every=4), pairs=True, per_source=True)
                want.append(w)
                rpq.rpq_batch_add(b, nfa, s, pairs_capacity=max(1, w.count) if keys else None, per_source=True)
            for turn in range(2):
                rpq.rpq_batch_run(b)
                for i, w in enumerate(want):
                    got = rpq.rpq_batch_result(b, i)
                    assert (got.count, got.hash) == (w.count, w.hash), (width, keys, turn, queries[i][0])
                    assert torch.equal(got.per_source, w.per_source)
                    assert not keys or torch.equal(got.pairs, w.pairs)
            rpq.rpq_batch_destroy(b)
    g.close()


@pytest.mark.parametrize("m", [0, 1, 2047, 2048, 2049, 4095, 4096, 4097, 70_001])
def test_ingest_tiles(rpq, m):
    """Edge counts around the tiles of the sort and of the duplicate pass, half of the edges twice, built one
    after another and from two threads at once, so that blocks of a released graph come back."""
    import threading
    n, labels = 777, 5
    rng = np.random.default_rng(m)

    def one(seed, out):
        r = np.random.default_rng(seed)
        src, dst = r.integers(0, n, m).astype(np.uint32), r.integers(0, n, m).astype(np.uint32)
        lab = r.integers(0, labels, m).astype(np.uint8)
        half = m // 2
        src[:half], dst[:half], lab[:half] = src[m - half:], dst[m - half:], lab[m - half:]
        g = rpq.rpq_graph_create(src, lab, dst, n, labels, flags=rpq.RPQ_BUILD_IN_CSR)
        for reverse in (False, True):
            u, w = (dst, src) if reverse else (src, dst)
            e = np.unique(np.stack([u, lab, w], axis=1).astype(np.int64), axis=0)
            rows = e[:, 0] * labels + e[:, 1]
            ptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n * labels))])
            got_ptr, got_dst = (t.cpu().numpy() for t in rpq.rpq_graph_export_csr(g, reverse))
            out.append(np.array_equal(got_ptr, ptr) and np.array_equal(got_dst, e[:, 2]))
        g.close()

    seeds = [int(x) for x in rng.integers(0, 1 << 30, 6)]
    print("case: %d edges" % m, flush=True)
    for s in seeds[:2]:
        one(s, out := [])
        assert out == [True, True]
    outs = [[], []]
    threads = [threading.Thread(target=lambda i=i: [one(s, outs[i]) for s in seeds[2 + 2 * i:4 + 2 * i]])
               for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert outs == [[True] * 4, [True] * 4]


@pytest.mark.parametrize("n_sources", [3, 64, 65, 600])
@pytest.mark.parametrize("opts", [None, dict(sync_every=2)])
def test_invalid_sources_leave_outputs_alone(rpq, n_sources, opts):
    """Ids out of order, twice, or beyond the graph: refused, with the caller's arrays as they were, also those
    of the sources without a first edge, whose results are written early; then a valid call."""
    import torch
    n = 6000
    src, lab, dst = hub_graph(n, [600, 17], 9000, seed=12)
    g = rpq.rpq_graph_create(src, lab, dst, n, 3, names=["a", "b", "c"])
    og = oracle.OracleGraph(n, src, lab, dst, 3, ["a", "b", "c"])
    good = np.unique(np.linspace(0, n - 1, n_sources).astype(np.uint32))
    for rx in ("a.b*.c", "c*", "a"):
        nfa = rpq.rpq_nfa_compile(rx, g.names)
        want = oracle.rpq(og, rx, sources=good)
        for how in ("order", "twice", "beyond"):
            bad = good.copy()
            if how == "order":
                bad[[0, -1]] = bad[[-1, 0]]
            elif how == "twice":
                bad[-1] = bad[-2]
            else:
                bad[-1] = n
            print("case: %d sources, %s, %s" % (len(good), rx, how), flush=True)
            per = torch.full((len(good), 2), -7, dtype=torch.int64, device="cuda")
            buf = torch.full((max(1, want.count),), -7, dtype=torch.int64, device="cuda")
            for keys in (None, buf):
                with pytest.raises(rpq.RpqError) as e:
                    rpq.rpq_eval(g, nfa, bad, opts=opts, pairs=keys, per_source=per)
                assert e.value.code == rpq.RPQ_EINVAL
                assert bool((per == -7).all()) and bool((buf == -7).all())
        same_as_oracle(evaluate(rpq, g, nfa, good, want, **(opts or {})), want)
    g.close()
