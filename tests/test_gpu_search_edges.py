"""GPU tests of calls at the edges of the search forms' dispatch: exactly the planned workspace, searches that
end or go on at the sizes where one form hands over to another, and the counts that describe a search.
Expected values come from the oracle or follow from how the graph is built."""
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


def say(*a):
    print("case:", *a, flush=True)


def u64(t):
    return t.cpu().numpy().view(np.uint64)


def same_as_oracle(got, want, keys=True):
    assert (got.count, got.hash, got.product_edges) == (want.count, want.hash, want.product_edges)
    assert np.array_equal(u64(got.per_source), want.per_source)
    if keys:
        assert np.array_equal(u64(got.pairs), want.pairs)


@pytest.mark.parametrize("n", [100, 1000, 3000])
@pytest.mark.parametrize("n_sources", [1, 9])
def test_sparse_runs_in_the_planned_workspace(rpq, n, n_sources):
    """The size that rpq_eval_workspace_size gives holds 2^15 triples, and these searches find fewer: closures
    where all triples together are fewer, chains of at most three edges elsewhere.  No call is refused."""
    import torch
    rng = np.random.default_rng(n)
    src, dst = rng.integers(0, n, 3 * n).astype(np.uint32), rng.integers(0, n, 3 * n).astype(np.uint32)
    lab = rng.integers(0, 2, 3 * n).astype(np.uint8)
    g = rpq.rpq_graph_create(src, lab, dst, n, 2, names=["a", "b"])
    og = oracle.OracleGraph(n, src, lab, dst, 2, ["a", "b"])
    s = np.unique(np.linspace(0, n - 1, n_sources).astype(np.uint32))
    for rx in ("a.b*", "a*.b?", "(a|b)*") if 3 * n * n_sources <= 1 << 15 else ("a.b", "a.b.a?", "a"):
        say(n, n_sources, rx)
        nfa = rpq.rpq_nfa_compile(rx, g.names)
        want = oracle.rpq(og, rx, sources=s)
        ws = torch.empty(rpq.rpq_eval_workspace_size(g, nfa, len(s), rpq.RPQ_SPARSE), dtype=torch.uint8, device="cuda")
        buf = torch.zeros(max(1, want.count), dtype=torch.int64, device="cuda")
        same_as_oracle(rpq.rpq_eval(g, nfa, s, flags=rpq.RPQ_SPARSE, pairs=buf, per_source=True, workspace=ws), want)
    g.close()


def test_sparse_levels_where_the_bitmaps_take_two_groups(rpq):
    """2^27 vertices and five states: the bitmaps of 300 sources take two units of 256, in flight one after the
    other, and count a level for each; the hash-set search counts the five frontiers once.  All vertices lie on
    a cycle, and vertex 0 also has edges to 70,000 others, so that the search passes 2^16 triples."""
    import torch
    n, hub = 1 << 27, 70_000
    free, _ = torch.cuda.mem_get_info()
    if free < 160 << 30:
        pytest.skip("needs 160 GB of free device memory")
    ring = torch.arange(n, dtype=torch.int32, device="cuda")
    src = torch.cat([ring, torch.zeros(hub, dtype=torch.int32, device="cuda")])
    dst = torch.cat([(ring + 1) % n, ring[1000:1000 + hub]])
    del ring
    lab = torch.zeros(src.numel(), dtype=torch.uint8, device="cuda")
    g = rpq.rpq_graph_create(src, lab, dst, n, 1, names=["a"])
    del src, dst, lab
    nfa = rpq.rpq_nfa_compile("a.a.a.a", g.names)
    s = np.arange(300, dtype=np.uint32) * 400_000
    need = rpq.rpq_eval_workspace_size(g, nfa, len(s), 0)
    say("workspace", need)
    assert need < 120 << 30
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    dense = rpq.rpq_eval(g, nfa, s, per_source=True, workspace=ws)
    got = rpq.rpq_eval(g, nfa, s, flags=rpq.RPQ_SPARSE, per_source=True, workspace=ws)
    # three more steps from each of the hub's 70,001 neighbours end at as many vertices
    assert (got.count, got.levels, got.max_depth) == (299 + 70_001, 5, 4)
    assert (got.hash, got.product_edges) == (dense.hash, dense.product_edges) and dense.levels == 10
    assert torch.equal(got.per_source, dense.per_source)
    g.close()
    del ws
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n_sources", [1, 64, 65, 700])
@pytest.mark.parametrize("form", ["bitmap", "levels", "sparse"])
def test_levels_of_searches_that_go_nowhere(rpq, n_sources, form):
    """One level where no source can leave (its frontier of zero-length walks), none where the automaton has no
    state to start in: however many sources there are and whichever form runs."""
    n = 9000
    src, dst = np.arange(100, 200, dtype=np.uint32), np.arange(200, 300, dtype=np.uint32)
    g = rpq.rpq_graph_create(src, np.zeros(100, dtype=np.uint8), dst, n, 1, names=["a"])
    s = np.arange(1000, 1000 + n_sources, dtype=np.uint32)
    kw = dict(flags=rpq.RPQ_SPARSE) if form == "sparse" else dict(opts=dict(sync_every=2)) if form == "levels" else {}
    for init, levels in ((1, 1), (0, 0)):
        nfa = rpq.rpq_nfa_compile("a.a", g.names)
        nfa.initial_mask = init
        say(n_sources, form, "initial states", init)
        r = rpq.rpq_eval(g, nfa, s, **kw)
        assert (r.count, r.levels, r.max_depth, r.product_edges) == (0, levels, 0, 0)
    g.close()


@pytest.mark.parametrize("n_sources", [600, 2500, 8192])
def test_units_of_graphs_below_8192_vertices(rpq, n_sources):
    """Five states on 8,192 vertices: too many rows for the search in LDS, units of 128 sources for 600 of them
    and wider ones for more."""
    n = 8192
    rng = np.random.default_rng(14)
    src, dst = rng.integers(0, n, 2 * n).astype(np.uint32), rng.integers(0, n, 2 * n).astype(np.uint32)
    lab = rng.integers(0, 3, 2 * n).astype(np.uint8)
    g = rpq.rpq_graph_create(src, lab, dst, n, 3, names=["a", "b", "c"])
    og = oracle.OracleGraph(n, src, lab, dst, 3, ["a", "b", "c"])
    s = np.unique(np.linspace(0, n - 1, n_sources).astype(np.uint32))
    for rx in ("(a|b)*.a.b", "(a.b?)*.c.a"):
        say(n_sources, rx)
        nfa = rpq.rpq_nfa_compile(rx, g.names)
        same_as_oracle(rpq.rpq_eval(g, nfa, s, per_source=True), oracle.rpq(og, rx, sources=s, pairs=False), keys=False)
    g.close()


@pytest.mark.parametrize("in_csr", [False, True])
def test_graph_holds_what_it_reports(rpq, in_csr):
    """2^25 edges of which 4,096 differ: the graph holds room for those alone, and device_bytes says so.  Three
    builds of another size let go of the blocks that the large one left behind; the device hands out memory in
    steps of up to 2 MiB."""
    import torch
    n, m = 4096, 1 << 25
    small = [torch.zeros(8, dtype=t, device="cuda") for t in (torch.int32, torch.uint8, torch.int32)]

    def settle():
        for _ in range(3):
            rpq.rpq_graph_create(*small, 8, 1).close()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]

    src = torch.arange(m, dtype=torch.int32, device="cuda") % n
    dst, lab = (src * 7 + 1) % n, torch.zeros(m, dtype=torch.uint8, device="cuda")
    before = settle()
    g = rpq.rpq_graph_create(src, lab, dst, n, 1, flags=rpq.RPQ_BUILD_IN_CSR if in_csr else 0)
    held, info = before - settle(), g.info()
    say("in_csr", in_csr, "held", held, "reported", info["device_bytes"])
    need = (1 + in_csr) * (4 * (n + 1) + 8 * n + 8 * n // 64 + 4 * n)
    assert info["n_edges"] == n and need <= info["device_bytes"] <= need + need // 8 + 4096
    assert held <= info["device_bytes"] + (4 << 20)
    for reverse in (False, True) if in_csr else (False,):
        ptr, nb = rpq.rpq_graph_export_csr(g, reverse)
        assert torch.equal(ptr, torch.arange(n + 1, dtype=torch.int32, device="cuda"))
        want = torch.empty(n, dtype=torch.int32, device="cuda")
        u, w = (dst[:n], src[:n]) if reverse else (src[:n], dst[:n])
        want[u.long()] = w
        assert torch.equal(nb, want)
    g.close()


@pytest.mark.parametrize("width", [128, 512])
def test_batch_levels_do_not_vary(rpq, width):
    """16,384 sources that all meet the same hub first, each with a chain of its own length: a unit takes as many
    levels as its longest chain, so the sum over the units tells which sources they hold.  Sources that meet the
    same hub stay in ascending order."""
    n_src, hub = 16384, 16384
    rng = np.random.default_rng(18)
    chain = rng.integers(1, 40, n_src)
    # chain cells after the hub and its 100 neighbours
    first = hub + 101 + np.concatenate([[0], np.cumsum(chain)[:-1]])
    n = int(hub + 101 + chain.sum())
    src = [np.arange(n_src), np.full(100, hub), np.arange(n_src)]
    dst = [np.full(n_src, hub), np.arange(hub + 1, hub + 101), first]
    cells = np.setdiff1d(np.arange(hub + 101, n), first + chain - 1)   # the last cell of a chain has no edge
    src, dst = np.concatenate(src + [cells]).astype(np.uint32), np.concatenate(dst + [cells + 1]).astype(np.uint32)
    g = rpq.rpq_graph_create(src, np.zeros(len(src), dtype=np.uint8), dst, n, 1, names=["a"])
    nfa = rpq.rpq_nfa_compile("a*", g.names)
    # depth of a source: its chain, or the two steps to a neighbour of the hub; a level for the seeds
    depth = np.maximum(chain, 2)
    want = int((depth.reshape(-1, width).max(axis=1) + 1).sum())
    for turn in range(4):
        b = rpq.rpq_batch_create(g, dict(batch_width=width, list_share=1))
        rpq.rpq_batch_add(b, nfa, np.arange(n_src, dtype=np.uint32), per_source=True)
        for run in range(3):
            rpq.rpq_batch_run(b)
            r = rpq.rpq_batch_result(b, 0)
            say("width", width, "turn", turn, run, "levels", r.levels, "expected", want)
            assert r.levels == want and r.count == n_src * 102 + int(chain.sum())
        rpq.rpq_batch_destroy(b)
    g.close()


def test_autotune_times_whole_segments(rpq):
    """One slot of 64 sources takes four units as its prefix of the queue, 256 of 8,192 sources.  The 4,096 that are
    prepared together run together, and no others: a candidate is scored by the sources that it ran."""
    n = 10_000
    src = np.arange(n, dtype=np.uint32)
    g = rpq.rpq_graph_create(src, np.zeros(n, dtype=np.uint8), (src * 7 + 3) % n, n, 1, names=["a"])
    b = rpq.rpq_batch_create(g)
    nfa = rpq.rpq_nfa_compile("a.a", g.names)
    rpq.rpq_batch_add(b, nfa, np.arange(8192, dtype=np.uint32), per_source=True)
    best = rpq.rpq_batch_autotune(b, [dict(batch_width=64, slots=1)])
    ran = b.outputs[0][1][:, 0].cpu().numpy()
    say("sources with a result", int((ran != 0).sum()))
    assert best["batch_width"] == 64 and ran[:4096].all() and not ran[4096:].any()
    rpq.rpq_batch_run(b)
    assert rpq.rpq_batch_result(b, 0).count == 8192
    rpq.rpq_batch_destroy(b)
    g.close()


def test_served_conjunctive_queries_pass_waiting_slices(rpq):
    """Two workers, eight slices of 4,096 sources and then a conjunctive query, with room for all of them at once:
    the query takes the first worker that comes free while a slice runs on the other, not the last one.  Every
    result is what it is alone."""
    import synth
    el = synth.workload_graph("rmat18_l8")
    g = rpq.rpq_graph_create(el.src, el.label, el.dst, el.n_vertices, el.n_labels, flags=rpq.RPQ_BUILD_IN_CSR,
                             names=el.names)
    nfa = rpq.rpq_nfa_compile("(a.b)*", el.names)
    slices = [np.arange(i * 4096, (i + 1) * 4096, dtype=np.uint32) for i in range(8)]
    alone = [rpq.rpq_eval(g, nfa, s) for s in slices]
    atoms, bind = [(0, "g.h?", 1), (1, "h", 2)], [int(el.src[np.argmax(el.label == 6)]), None, None]
    want = rpq.crpq_eval(g, atoms, 3, binding=bind)
    srv = rpq.Server(g, 24 << 30, workers=2)
    warm = [srv.submit_rpq(nfa, slices[0]), srv.submit_crpq(atoms, 3, binding=bind)]
    for t in warm:
        srv.wait(t)
    tickets = [srv.submit_rpq(nfa, s) for s in slices]
    last = srv.submit_crpq(atoms, 3, binding=bind)
    done = [srv.wait(t) for t in tickets]
    x = srv.wait(last)
    before = sum(d["start_ms"] < x["start_ms"] for d in done)
    say("slices that began before the query", before, "wait", x["start_ms"] - x["arrival_ms"])
    srv.stop()
    assert (x["status"], x["count"], x["hash"]) == (0, want.count, want.hash)
    for d, a in zip(done, alone):
        assert (d["status"], d["count"], d["hash"], d["product_edges"]) == (0, a.count, a.hash, a.product_edges)
    assert before <= 4
    g.close()


def test_edge_scan_leaves_only_its_pairs_in_the_workspace(rpq):
    """All edges of one label as a query: the scan's offsets (8 bytes a source) do not stay beside the pairs, so
    7.9 MB are enough where 7.7 are needed."""
    import torch
    n, m = 100_000, 800_000
    rng = np.random.default_rng(n)
    src, lab, dst = (rng.integers(0, n, m).astype(np.uint32), rng.integers(0, 4, m).astype(np.uint8),
                     rng.integers(0, n, m).astype(np.uint32))
    g = rpq.rpq_graph_create(src, lab, dst, n, 4, names=["a", "b", "c", "d"])
    want = len(np.unique(src[lab == 0].astype(np.uint64) << np.uint64(32) | dst[lab == 0]))
    ws = 7_900_000
    r = rpq.crpq_eval(g, [(0, "a", 1)], 2, workspace_bytes=ws)
    held = g.workspace(256).numel()   # the binding grows it when the library asks for more
    say("workspace", held)
    assert r.count == want and held == ws
    g.close()


@pytest.fixture(scope="module")
def ranked(rpq):
    """300,000 vertices of which a label leads to a fifth at most: above 64 MB of bitmaps (9,000 sources) a state
    has rows only for those."""
    n, m = 300_000, 240_000
    rng = np.random.default_rng(31)
    src, dst = rng.integers(0, n, m).astype(np.uint32), rng.integers(0, n, m).astype(np.uint32)
    lab = rng.choice(4, size=m, p=[0.3, 0.3, 0.3, 0.1]).astype(np.uint8)
    dst[lab == 3] = dst[lab == 3] % 1000
    names = ["a", "b", "c", "d"]
    g = rpq.rpq_graph_create(src, lab, dst, n, 4, flags=rpq.RPQ_BUILD_IN_CSR, names=names)
    yield (g, oracle.OracleGraph(n, src, lab, dst, 4, names), oracle.OracleGraph(n, dst, lab, src, 4, names),
           np.unique(rng.integers(0, n, 9000)).astype(np.uint32), rng)
    g.close()


@pytest.mark.parametrize("reverse", [False, True])
@pytest.mark.parametrize("rx,back", [("a.b*.c", "c.b*.a"), ("(a|d)?.c", "c.(a|d)?"), ("d?", "d?")])
def test_ranked_rows_keys_streams_and_noalloc(rpq, ranked, rx, back, reverse):
    g, og, ogt, s, _ = ranked
    nfa = rpq.rpq_nfa_compile(rx, g.names)
    want = oracle.rpq(ogt if reverse else og, back if reverse else rx, sources=s)
    flags = rpq.RPQ_REVERSE if reverse else 0
    say(rx, "reverse", reverse, "keys", want.count)
    got = rpq.rpq_eval(g, nfa, s, flags=flags, pairs=True, per_source=True)
    assert (got.count, got.hash) == (want.count, want.hash)
    assert np.array_equal(u64(got.pairs), want.pairs) and np.array_equal(u64(got.per_source), want.per_source)
    if not reverse:   # a reversed automaton counts its own product edges
        assert got.product_edges == want.product_edges
    chunks = []
    st = rpq.rpq_eval_stream(g, nfa, lambda k: chunks.append(k.copy()) and None, s, flags=flags, chunk_keys=1000,
                             per_source=True)
    assert (st.count, st.hash, st.written) == (want.count, want.hash, want.count)
    assert np.array_equal(np.concatenate(chunks), want.pairs) and np.array_equal(u64(st.per_source), want.per_source)
    na = rpq.rpq_eval_noalloc(g, nfa, s, flags=flags)
    assert (na.count, na.hash, na.product_edges) == (got.count, got.hash, got.product_edges)


@pytest.mark.parametrize("rx", ["a.b*.c", "(a|d)?.c", "a.b"])
def test_ranked_rows_with_a_destination_filter(rpq, ranked, rx):
    """A bit-parallel atom from 9,000 sources whose destinations are limited to a tenth of the vertices."""
    g, og, _, s, rng = ranked
    keep = np.unique(rng.integers(0, og.n_vertices, og.n_vertices // 10)).astype(np.uint32)
    keys = oracle.rpq(og, rx, sources=s).pairs
    keys = keys[np.isin((keys & np.uint64(0xFFFFFFFF)).astype(np.uint32), keep)]
    want = np.stack([(keys >> np.uint64(32)).astype(np.uint32), (keys & np.uint64(0xFFFFFFFF)).astype(np.uint32)], axis=1)
    r = rpq.crpq_eval(g, [(0, rx, 1)], 2, domain=[s, keep], tuples=True,
                      flags=rpq.CRPQ_FORCE_DENSE | rpq.CRPQ_NO_EDGE_SCAN | rpq.CRPQ_NO_REVERSE)
    say(rx, "tuples", len(want))
    assert len(want) > 10 and r.count == len(want) and r.atom_strategy[0] & 0xFF == 2
    assert np.array_equal(r.tuples.cpu().numpy().view(np.uint32), want)


@pytest.mark.parametrize("form", ["bitmap", "hash set"])
@pytest.mark.parametrize("past", [0, 1])
def test_sparse_search_at_its_limit(rpq, form, past):
    """2^16 triples are found by the sparse search itself, one more by the bit-parallel one (whose level kernels the
    profile counts).  A bitmap of one source is small; one of 512 sources and 600,000 vertices passes 64 MB."""
    n = 70_000 if form == "bitmap" else 600_000
    s = np.arange(1 if form == "bitmap" else 512, dtype=np.uint32)
    leaves = (1 << 16) - len(s) + past   # a triple for every seed, one for every edge of vertex 0
    src, dst = np.zeros(leaves, dtype=np.uint32), np.arange(1000, 1000 + leaves, dtype=np.uint32)
    lab = np.zeros(leaves, dtype=np.uint8)
    g = rpq.rpq_graph_create(src, lab, dst, n, 1, names=["a"])
    want = oracle.rpq(oracle.OracleGraph(n, src, lab, dst, 1, ["a"]), "a", sources=s)
    nfa = rpq.rpq_nfa_compile("a", g.names)
    rpq.rpq_profile_enable(True)
    rpq.rpq_profile_read(reset=True)
    got = rpq.rpq_eval(g, nfa, s, flags=rpq.RPQ_SPARSE, pairs=True, per_source=True)
    prof = rpq.rpq_profile_read(reset=True)
    rpq.rpq_profile_enable(False)
    say(form, leaves, "level launches", prof["expand_launches"])
    same_as_oracle(got, want)
    assert (prof["expand_launches"] > 0) == (past == 1) and (got.levels, got.max_depth) == (2, 1)
    g.close()


def test_sparse_workspace_asks_for_more(rpq):
    """Where the bit-parallel search may not take over, because there are too many sources or its bitmaps do not
    fit, a search that outgrows its workspace names a larger one; the binding's own grows until it ends."""
    import torch
    n = 8000
    rng = np.random.default_rng(5)
    src, dst = rng.integers(0, n, 2 * n).astype(np.uint32), rng.integers(0, n, 2 * n).astype(np.uint32)
    lab = rng.integers(0, 2, 2 * n).astype(np.uint8)
    g = rpq.rpq_graph_create(src, lab, dst, n, 2, names=["a", "b"])
    og = oracle.OracleGraph(n, src, lab, dst, 2, ["a", "b"])
    nfa = rpq.rpq_nfa_compile("(a|b)*", g.names)
    s = np.unique(np.linspace(0, n - 1, 600).astype(np.uint32))
    want = oracle.rpq(og, "(a|b)*", sources=s)
    same_as_oracle(rpq.rpq_eval(g, nfa, s, flags=rpq.RPQ_SPARSE, pairs=True, per_source=True), want)
    held = g.workspace(256).numel()
    say("workspace", held, "for", want.count, "keys")
    assert held > 64 << 20
    g.close()
    n = 200_000   # bitmaps of 25 MB and more: not in the 1.7 MB planned for the search
    src, dst = rng.integers(0, n, 3 * n).astype(np.uint32), rng.integers(0, n, 3 * n).astype(np.uint32)
    lab = np.zeros(3 * n, dtype=np.uint8)
    g = rpq.rpq_graph_create(src, lab, dst, n, 1, names=["a"])
    og = oracle.OracleGraph(n, src, lab, dst, 1, ["a"])
    nfa = rpq.rpq_nfa_compile("a*", g.names)
    s = np.arange(3, dtype=np.uint32)
    want = oracle.rpq(og, "a*", sources=s)
    buf = torch.zeros(want.count, dtype=torch.int64, device="cuda")
    ws = torch.empty(rpq.rpq_eval_workspace_size(g, nfa, len(s), rpq.RPQ_SPARSE), dtype=torch.uint8, device="cuda")
    with pytest.raises(rpq.RpqError) as e:
        rpq.rpq_eval(g, nfa, s, flags=rpq.RPQ_SPARSE, pairs=buf, per_source=True, workspace=ws)
    assert e.value.code == rpq.RPQ_ENOMEM
    same_as_oracle(rpq.rpq_eval(g, nfa, s, flags=rpq.RPQ_SPARSE, pairs=buf, per_source=True), want)
    g.close()


@pytest.mark.parametrize("keys", [True, False])
@pytest.mark.parametrize("width", [0, 64, 1024])
def test_batch_segments_against_the_oracle(rpq, width, keys):
    """Queries of 4,095 to 4,097 sources (a block prepares 4,096), of sources without a first edge alone, and with
    the empty word."""
    n = 5000
    rng = np.random.default_rng(10)
    hubs = [(0, 600), (1, 3000), (2, 17)]
    src = np.concatenate([np.full(d, h) for h, d in hubs] + [rng.integers(0, 3500, 6000)]).astype(np.uint32)
    dst, lab = rng.integers(0, n, len(src)).astype(np.uint32), rng.integers(0, 3, len(src)).astype(np.uint8)
    g = rpq.rpq_graph_create(src, lab, dst, n, 3, names=["a", "b", "c"])
    og = oracle.OracleGraph(n, src, lab, dst, 3, ["a", "b", "c"])
    queries = [(rx, np.arange(k, dtype=np.uint32)) for k in (4095, 4096, 4097) for rx in ("a.b*.c", "(a.b)*")]
    queries += [("c.a", np.arange(3500, 4200, dtype=np.uint32)), ("c?", np.arange(3400, 4300, dtype=np.uint32))]
    b = rpq.rpq_batch_create(g, dict(batch_width=width) if width else None)
    want = [oracle.rpq(og, rx, sources=s) for rx, s in queries]
    for (rx, s), w in zip(queries, want):
        rpq.rpq_batch_add(b, rpq.rpq_nfa_compile(rx, g.names), s, pairs_capacity=max(1, w.count) if keys else None,
                          per_source=True)
    for turn in range(2):
        rpq.rpq_batch_run(b)
        for i, w in enumerate(want):
            say("width", width, "keys", keys, "run", turn, queries[i][0], len(queries[i][1]))
            same_as_oracle(rpq.rpq_batch_result(b, i), w, keys)
    rpq.rpq_batch_destroy(b)
    g.close()


@pytest.mark.parametrize("rx", ["a", "a.b", "a.b?.c", "(a|b).c.(a.b)?", "a?", "a*.b"])
@pytest.mark.parametrize("bound", [None, 0, 1, 2])
def test_sparse_search_of_finite_languages(rpq, rx, bound):
    """The sparse search launches no level that the automaton's longest walk cannot reach: results, levels and product
    edges as the oracle and the bit-parallel search have them, with bounds below and above that walk."""
    n = 400
    rng = np.random.default_rng(21)
    src, dst, lab = (rng.integers(0, k, 1500) for k in (n, n, 3))
    g = rpq.rpq_graph_create(src.astype(np.uint32), lab.astype(np.uint8), dst.astype(np.uint32), n, 3, names=["a", "b", "c"])
    og = oracle.OracleGraph(n, src, lab, dst, 3, ["a", "b", "c"])
    nfa = rpq.rpq_nfa_compile(rx, g.names)
    for s in (np.arange(1, dtype=np.uint32), np.arange(0, n, 2, dtype=np.uint32)):
        say(rx, "bound", bound, "sources", len(s))
        want = oracle.rpq(og, rx, sources=s, max_length=bound)
        level = rpq.rpq_eval(g, nfa, s, opts=dict(sync_every=1), max_length=bound)
        got = rpq.rpq_eval(g, nfa, s, flags=rpq.RPQ_SPARSE, pairs=True, per_source=True, max_length=bound)
        same_as_oracle(got, want)
        assert (got.max_depth, got.levels) == (level.max_depth, level.max_depth + 1)
    g.close()
