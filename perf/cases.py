"""The work that users of this framework have it do, as cases that can be timed and compared.

Each case is one call (or one build-and-export) through the public entry points on a seeded graph drawn
on the GPU: R-MAT graphs with Zipf edge labels, a uniform graph, and the typed social graph of the
conjunctive queries.  Every output is a whole number or a set of keys or tuples, so outputs are equal
or wrong.  `levels` is left out of them: it counts the rounds of every group of units and so describes
the plan, not the result.
"""
import math

import numpy as np
import torch

import paper_2602_20748_amd as rpq

NAMES = [chr(ord("a") + i) for i in range(16)]
# the query shapes of the benchmark and its generated mixes: closures, prefixes, unions, alternating
# closures, plain chains
SHAPES = ["a*", "a.b*", "(a|b).c*", "a.b*.c", "(a.b)*", "a.b.c*", "a?.b*", "a.b.c.d", "(a|b|c).d*", "b.(a|c)*",
          "c.d?.a+", "a.(b.c)*.d?"]
SHAPE_STATES = [2, 3, 4, 4, 3, 4, 3, 5, 5, 4, 4, 5]   # one more than the label occurrences
KNOWS_CYCLE, PROPAGATION = "cycle", "propagation"


def listed():
    ev = dict(kind="eval", form="dense", reverse=False, bound=-1)
    return [
        # the smallest whole evaluation: all pairs with keys on 1,000 vertices, bound by launches and waits
        dict(ev, name="uniform_pairs", graph="uniform", vertices=1000, edges=5000, labels=4, query="a.b.c*",
             pick="all", sources=1000, out="keys"),
        # an interactive question: what does one vertex reach, with the keys
        dict(ev, name="single_dense", graph="rmat", scale=18, labels=8, query="a.b*", pick="start", sources=1,
             out="keys"),
        # the same on a graph of four million vertices through the hash-set search, as serving workers run it
        dict(ev, name="single_sparse", graph="rmat", scale=22, labels=16, query="b.(a|c)*", pick="start", sources=1,
             out="keys", form="sparse"),
        # who reaches these, in at most three steps: in-edges, reversed automaton, ragged source count
        dict(ev, name="reverse_bounded", graph="rmat", scale=20, labels=8, query="(a|b|c).d*", pick="sampled",
             sources=1003, out="per_source", reverse=True, bound=3),
        # a slice of sources with every result key wanted: bound by writing the keys
        dict(ev, name="slice_pairs", graph="rmat", scale=18, labels=8, query="(a|b).c*", pick="slice", sources=2500,
             out="keys"),
        # the served slice: 4,096 consecutive sources of a large graph, tallies per source
        dict(ev, name="slice_per_source", graph="rmat", scale=22, labels=16, query="a.b*.c", pick="slice",
             sources=4096, out="per_source"),
        # all pairs of a graph of 262,144 vertices, counted and checksummed: many units in flight
        dict(ev, name="all_pairs", graph="rmat", scale=18, labels=8, query="(a.b)*", pick="all", sources=1 << 18,
             out="count"),
        # the benchmark's headline shape: the largest graph, 65,536 sampled sources
        dict(ev, name="sampled_large", graph="rmat", scale=23, labels=16, query="a.b*", pick="sampled",
             sources=65536, out="count"),
        # many small questions answered together by the batched persistent launch
        dict(name="batch_single", kind="batch", scale=18, labels=8, singles=256, slices=0, width=0, slice=0),
        # a mixed batch: single sources beside slices
        dict(name="batch_mixed", kind="batch", scale=20, labels=16, singles=32, slices=32, width=1024, slice=2048),
        # the information-propagation join over messages, creators, tags and reply chains, tuples wanted
        dict(name="crpq_propagation", kind="crpq", shape=PROPAGATION, persons=400_000, messages=4_000_000, tags=16384,
             sample=0),
        # loading a graph in both directions, up to its exported adjacency
        dict(name="ingest", kind="ingest", scale=20, labels=8),
    ]


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.6:
        i = rng.randrange(len(SHAPES))
        scale = rng.randint(12, 22)
        c = dict(kind="eval", form="dense", graph="rmat", scale=scale, labels=rng.choice([4, 8, 16]), query=SHAPES[i],
                 pick=rng.choice(["slice", "sampled", "sampled", "start"]), out=rng.choice(["keys", "per_source", "count"]),
                 reverse=rng.random() < 0.25, bound=rng.choice([-1, -1, -1, 2, 5]))
        # rows of states x vertices x sources well below the largest listed case's; keys fit a buffer
        most = min(1 << scale, (1 << 38) // (SHAPE_STATES[i] << scale))
        if c["out"] == "keys":
            most = min(most, (1 << 29) >> scale)
        c["sources"] = _log(rng, 1, max(1, most))
        if rng.random() < 0.2:
            c.update(form="sparse", sources=min(c["sources"], rng.randint(1, 8)), pick="start")
        return c
    if u < 0.75:
        scale = rng.randint(14, 20)
        return dict(kind="batch", scale=scale, labels=rng.choice([8, 16]), singles=_log(rng, 8, 256),
                    slices=rng.randint(0, 24), width=rng.choice([0, 256, 1024, 2048]), slice=_log(rng, 64, 2048))
    if u < 0.88:
        shape = rng.choice([KNOWS_CYCLE, PROPAGATION])
        persons = _log(rng, 5_000, 300_000)
        return dict(kind="crpq", shape=shape, persons=persons, messages=persons * rng.randint(5, 10),
                    tags=_log(rng, 100, 16384), sample=rng.randint(16, 160) if shape == KNOWS_CYCLE else 0)
    return dict(kind="ingest", scale=rng.randint(12, 20), labels=rng.choice([1, 4, 8, 16]))


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------
def _zipf_cdf(n, s):
    w = torch.arange(1, n + 1, dtype=torch.float64) ** -s
    return (torch.cumsum(w, 0) / w.sum()).to(torch.float32).cuda()


def _pick_by(cdf, n, gen):
    u = torch.rand(n, generator=gen, device="cuda")
    return torch.searchsorted(cdf, u).clamp_(max=cdf.numel() - 1)


def _rmat(scale, n_labels, gen):
    """R-MAT (0.57, 0.19, 0.19, 0.05) with 16 edges a vertex, shuffled vertex ids, labels Zipf(1.1)."""
    n, m = 1 << scale, 16 << scale
    perm = torch.randperm(n, generator=gen, device="cuda").to(torch.int32)
    src = torch.empty(m, dtype=torch.int32, device="cuda")
    dst = torch.empty(m, dtype=torch.int32, device="cuda")
    label = torch.empty(m, dtype=torch.uint8, device="cuda")
    cdf = _zipf_cdf(n_labels, 1.1)
    for lo in range(0, m, 1 << 25):
        k = min(m, lo + (1 << 25)) - lo
        s = torch.zeros(k, dtype=torch.int32, device="cuda")
        d = torch.zeros(k, dtype=torch.int32, device="cuda")
        for _ in range(scale):
            u = torch.rand(k, generator=gen, device="cuda")
            down = u >= 0.76
            s.mul_(2).add_(down)
            d.mul_(2).add_(((u >= 0.57) & ~down) | (u >= 0.95))
        src[lo:lo + k] = perm[s.long()]
        dst[lo:lo + k] = perm[d.long()]
        label[lo:lo + k] = _pick_by(cdf, k, gen).to(torch.uint8)
    return src, label, dst


def _uniform(n, m, n_labels, gen):
    key = torch.randperm(n * n * n_labels, generator=gen, device="cuda")[:m]
    return (key // (n * n_labels)).to(torch.int32), (key // n % n_labels).to(torch.uint8), (key % n).to(torch.int32)


def _social(P, M, T, gen):
    """Persons, messages and tags with knows (power law, both directions), hasCreator, replyOf (forest of
    geometric depth) and hasTag (one to three Zipf tags a message)."""
    def person(k):
        w = torch.arange(1, P + 1, dtype=torch.float64) ** (-1.0 / 1.5)
        cdf = (torch.cumsum(w, 0) / w.sum()).to(torch.float32).cuda()
        return _pick_by(cdf, k, gen)
    ids = torch.randperm(P, generator=gen, device="cuda")
    a, b = ids[person(10 * P)], ids[person(10 * P)]
    a, b = a[a != b], b[a != b]
    msg = torch.arange(P, P + M, device="cuda")
    creator = (torch.rand(M, generator=gen, device="cuda", dtype=torch.float64) * P).long()
    depth = (torch.log1p(-torch.rand(M, generator=gen, device="cuda", dtype=torch.float64)) / math.log(0.7)).long()
    order = torch.argsort(depth, stable=True)
    first = torch.searchsorted(depth[order], torch.arange(int(depth.max()) + 2, device="cuda"))
    above = depth[order] > 0
    d = depth[order][above]
    size = first[d] - first[d - 1]
    parent = order[first[d - 1] + (torch.rand(d.numel(), generator=gen, device="cuda", dtype=torch.float64) * size).long()]
    child, keep = order[above], size > 0
    n_tags = torch.randint(1, 4, (M,), generator=gen, device="cuda")
    cdf = _zipf_cdf(T, 1.2)
    tag_src, tag_dst = [], []
    for i in range(3):
        has = n_tags > i
        tag_src.append(msg[has])
        tag_dst.append(P + M + _pick_by(cdf, M, gen)[has])
    parts = [(a, b), (b, a), (msg, creator), (P + child[keep], P + parent[keep])] + list(zip(tag_src, tag_dst))
    src = torch.cat([x for x, _ in parts]).to(torch.int32)
    dst = torch.cat([y for _, y in parts]).to(torch.int32)
    label = torch.cat([torch.full((x.numel(),), l, dtype=torch.uint8, device="cuda")
                       for (x, _), l in zip(parts, [0, 0, 1, 2, 3, 3, 3])])
    kind = torch.cat([torch.full((k,), l, dtype=torch.uint8, device="cuda") for k, l in ((P, 0), (M, 1), (T, 2))])
    return src, label, dst, kind


def _sources(case, V, src, label, gen):
    n = case["sources"]
    if case["pick"] == "all":
        return None
    if case["pick"] == "slice":
        lo = int(torch.randint(0, V - n + 1, (1,), generator=gen, device="cuda"))
        return torch.arange(lo, lo + n, dtype=torch.int32, device="cuda")
    if case["pick"] == "start":   # vertices that have an edge of the query's first label to leave by
        pool = src[label == NAMES.index(next(x for x in case["query"] if x in NAMES))]
        picked = pool[torch.randint(0, pool.numel(), (n,), generator=gen, device="cuda")]
    else:
        picked = torch.randperm(V, generator=gen, device="cuda")[:n].to(torch.int32)
    return torch.unique(picked)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "crpq":
        P, M, T = case["persons"], case["messages"], case["tags"]
        src, label, dst, vl = _social(P, M, T, gen)
        g = rpq.rpq_graph_create(src, label, dst, P + M + T, 4, vertex_label=vl, flags=rpq.RPQ_BUILD_IN_CSR,
                                 names=["knows", "hasCreator", "replyOf", "hasTag"])
        if case["shape"] == KNOWS_CYCLE:
            n = case["sample"] ** 3
            people = torch.randperm(P, generator=gen, device="cuda")[:case["sample"]].sort().values.to(torch.int32)
            return dict(case=case, g=g, n_vars=3, atoms=[(0, "knows.knows*", 1), (1, "knows.knows*", 2), (2, "knows.knows*", 0)],
                        tuples=torch.zeros((n, 3), dtype=torch.int32, device="cuda"),
                        kw=dict(domain=[people] * 3, vertex_label=[0] * 3, capacity=n))
        return dict(case=case, g=g, n_vars=4, atoms=[(0, "hasTag", 1), (0, "hasCreator", 2), (0, "replyOf*", 3)],
                    tuples=torch.zeros((2 * M, 3), dtype=torch.int32, device="cuda"),
                    kw=dict(binding=[None, P + M, None, None], vertex_label=[1, 2, 0, 1], capacity=2 * M))
    L = case["labels"]
    if kind == "eval" and case["graph"] == "uniform":
        V = case["vertices"]
        src, label, dst = _uniform(V, case["edges"], L, gen)
    else:
        V = 1 << case["scale"]
        src, label, dst = _rmat(case["scale"], L, gen)
    if kind == "ingest":
        return dict(case=case, edges=(src, label, dst), V=V,
                    adjacency=[torch.zeros(src.numel(), dtype=torch.int32, device="cuda") for _ in range(2)])
    reverse = kind == "eval" and case["reverse"]
    g = rpq.rpq_graph_create(src, label, dst, V, L, flags=rpq.RPQ_BUILD_IN_CSR if reverse else 0, names=NAMES[:L])
    if kind == "batch":
        b = rpq.rpq_batch_create(g, dict(batch_width=case["width"]) if case["width"] else None)
        n_slices = V // case["slice"] if case["slice"] else 1
        lows = torch.randint(0, n_slices, (case["slices"],), generator=gen, device="cuda").tolist()
        ones = torch.randint(0, V, (case["singles"],), generator=gen, device="cuda", dtype=torch.int32)
        for i in range(case["singles"]):
            rpq.rpq_batch_add(b, rpq.rpq_nfa_compile(SHAPES[i % len(SHAPES)], g.names), ones[i:i + 1].clone())
        for i, k in enumerate(lows):
            s = torch.arange(k * case["slice"], (k + 1) * case["slice"], dtype=torch.int32, device="cuda")
            rpq.rpq_batch_add(b, rpq.rpq_nfa_compile(SHAPES[i % len(SHAPES)], g.names), s, per_source=True)
        return dict(case=case, g=g, b=b, n=case["singles"] + case["slices"])
    st = dict(case=case, g=g, nfa=rpq.rpq_nfa_compile(case["query"], g.names), pairs=None, per_source=None)
    st["sources"] = _sources(case, V, src, label, gen)
    n = V if st["sources"] is None else st["sources"].numel()
    if case["out"] == "keys":
        st["pairs"] = torch.zeros(max(n * V // 6, min(n * V, 1 << 20)), dtype=torch.int64, device="cuda")
    if case["out"] == "per_source":
        st["per_source"] = torch.zeros((n, 2), dtype=torch.int64, device="cuda")
    return st


# ------------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------------
# Results of a size that only the search knows go into a buffer that the program keeps, zero past their end.
def _signed(x):
    return x - (1 << 64) if x >> 63 else x


def run(state):
    case = state["case"]
    if case["kind"] == "eval":
        r = rpq.rpq_eval(state["g"], state["nfa"], state["sources"],
                         flags=(rpq.RPQ_REVERSE if case["reverse"] else 0) | (rpq.RPQ_SPARSE if case["form"] == "sparse" else 0),
                         pairs=state["pairs"], per_source=state["per_source"],
                         max_length=case["bound"] if case["bound"] >= 0 else None, allow_overflow=True)
        out = [r.count, _signed(r.hash), r.product_edges, r.max_depth]
        return out + [x for x in (state["pairs"], r.per_source) if x is not None]
    if case["kind"] == "batch":
        b = state["b"]
        b.run()
        res = [b.result(i) for i in range(state["n"])]
        out = [np.array([[r.count, _signed(r.hash), r.product_edges] for r in res], dtype=np.int64)]
        return out + [r.per_source for r in res if r.per_source is not None]
    if case["kind"] == "crpq":
        r = rpq.crpq_eval(state["g"], state["atoms"], state["n_vars"], tuples=True, allow_overflow=True, **state["kw"])
        state["tuples"][:r.written].copy_(r.tuples)
        return [r.count, _signed(r.hash), state["tuples"]]
    src, label, dst = state["edges"]
    g = rpq.rpq_graph_create(src, label, dst, state["V"], case["labels"], flags=rpq.RPQ_BUILD_IN_CSR,
                             names=NAMES[:case["labels"]])
    out = []
    for reverse, adjacency in zip((False, True), state["adjacency"]):
        row_ptr, neighbours = rpq.rpq_graph_export_csr(g, reverse=reverse)
        adjacency[:neighbours.numel()].copy_(neighbours)
        out += [row_ptr, adjacency]
    g.close()
    return out


def exact(case, seed):
    """The exported adjacency, by sorting the edge list's distinct triples.  Everything else is a search's
    result: whole numbers and keys with nothing to round."""
    if case["kind"] != "ingest":
        return None
    src, label, dst = prepare(case, seed)["edges"]
    V, L = 1 << case["scale"], case["labels"]
    out = []
    for a, b in ((src, dst), (dst, src)):
        key = torch.unique((a.long() * L + label.long()) * V + b.long())
        ends = torch.arange(V * L + 1, device="cuda") * V
        out += [torch.searchsorted(key, ends).to(torch.int32), torch.zeros_like(a)]
        out[-1][:key.numel()] = (key % V).to(torch.int32)
    return out


def work(case):
    """Each edge and row pointer read once, each result written once.  How many keys a search finds is not
    known before it ran: they are counted as one for every fourth of its (source, vertex) pairs, which is
    near what the closures of an R-MAT graph give.  Nothing is a floating-point operation; an operation here
    is the checksum of one key or tuple (about twenty integer operations)."""
    kind = case["kind"]
    if kind == "crpq":
        P, M = case["persons"], case["messages"]
        rows = 3 * case["sample"] ** 3 if case["shape"] == KNOWS_CYCLE else 4 * M
        return dict(bytes=4 * (20 * P + 4 * M) + 4 * rows, flops=20.0 * rows)
    V = case["vertices"] if case.get("graph") == "uniform" else 1 << case["scale"]
    E = case["edges"] if case.get("graph") == "uniform" else 16 * V
    rows = 4 * V * case["labels"]   # the row pointers
    if kind == "ingest":
        return dict(bytes=9 * E + 2 * (4 * E + rows), flops=0)
    if kind == "batch":
        n = case["singles"] + case["slices"] * case["slice"]
        return dict(bytes=4 * E + rows + 16 * case["slices"] * case["slice"], flops=20.0 * n * V / 4)
    keys = case["sources"] * V / 4
    wrote = 8 * keys if case["out"] == "keys" else 16 * case["sources"] if case["out"] == "per_source" else 0
    return dict(bytes=4 * E + rows + wrote, flops=20.0 * keys)
