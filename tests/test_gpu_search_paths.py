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
