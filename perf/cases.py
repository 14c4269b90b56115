"""Cases that the framework's speed is measured on: the calls a program that uses it makes.

Four families, each through the entry points of ``paper_2512_02278_amd.ann``:

``search``   ``ann_search`` on an index resident on the GPU: routing, execution order, beam search.
``route``    ``ann_route``: the routing alone, as a pipeline that overlaps it with the search issues it.
``combine``  ``ann_merge_topk`` and ``ann_gather_vectors``: the candidates that came back from several partitions
             are merged, and the vectors of the merged lists are fetched.
``build``    ``ann_graph_optimize``: kNN lists into a search graph.

Element types, metrics, row lengths, degrees, list sizes, widths, entry rules and batch sizes are those of the
repository's benchmark, tests and smoke configuration.  The indices are smaller than the benchmark's largest (an index of
100 million vectors takes minutes to make); clusters hold about as many vectors, and batches about as many queries per
cluster, as there.
"""
import torch

from paper_2512_02278_amd import ann, inputs

DEVICE = "cuda"
DTYPES = {"u8": torch.uint8, "f16": torch.float16, "f32": torch.float32}
SIZES = {"u8": 1, "f16": 2, "f32": 4}
METRICS = {"l2": ann.ANN_L2, "ip": ann.ANN_IP}


# ------------------------------------------------------------------------------------------------ the cases


def _search(dtype, dim, n, clusters, degree, nq, k, itopk, width, iters, metric="l2", entry="routed", route_c=1, n_entry=32):
    return dict(kind="search", dtype=dtype, dim=dim, n=n, clusters=clusters, degree=degree, nq=nq, k=k, itopk=itopk,
                width=width, iters=iters, metric=metric, entry=entry, route_c=route_c, n_entry=n_entry)


def _route(dtype, dim, clusters, nq, route_c, metric="l2"):
    return dict(kind="route", dtype=dtype, dim=dim, clusters=clusters, nq=nq, route_c=route_c, metric=metric)


def _combine(dtype, dim, n, nq, parts, k):
    return dict(kind="combine", dtype=dtype, dim=dim, n=n, nq=nq, parts=parts, k=k)


def _build(n, clusters, d_in, d_out):
    return dict(kind="build", n=n, clusters=clusters, d_in=d_in, d_out=d_out)


def listed():
    return [
        # the smoke configuration: a handful of interactive queries on a small index, where latency and launches count
        dict(_search("u8", 128, 10_000, 100, 32, 100, 10, 64, 1, 50), name="search_u8_10k_batch100"),
        # a serving batch on the one-million index of the benchmark
        dict(_search("u8", 128, 1_000_000, 1000, 32, 10_000, 10, 128, 4, 100), name="search_u8_1m_batch10k"),
        # throughput: a batch with some sixty queries per cluster, as the benchmark's headline has; grouped execution order
        dict(_search("u8", 128, 16_000_000, 8192, 32, 500_000, 10, 184, 4, 200), name="search_u8_16m_batch500k"),
        # float image descriptors, degree 64, long candidate list
        dict(_search("f32", 96, 1_000_000, 410, 64, 20_000, 10, 256, 4, 150), name="search_f32_1m_batch20k"),
        # text embeddings, inner product, a hundred results per query
        dict(_search("f16", 768, 400_000, 164, 64, 5_000, 100, 256, 8, 200, metric="ip"), name="search_f16_768_400k_batch5k"),
        # no centroids: entries drawn over the whole index, visited set in the hash; odd degree, rows that leave lanes idle
        dict(_search("f16", 200, 200_003, 200, 27, 3_001, 7, 100, 3, 100, entry="uniform"), name="search_f16_200_uniform"),
        # stage 1 of a large batch against a large partition's centroids
        dict(_route("u8", 128, 16_384, 500_000, 1), name="route_u8_500k_16k"),
        dict(_route("f32", 96, 4_096, 100_000, 1), name="route_f32_100k_4k"),
        dict(_route("f16", 768, 8_192, 25_000, 4, metric="ip"), name="route_f16_25k_8k_top4"),
        # the origin's side of a batch that was sent to eight partitions
        dict(_combine("u8", 128, 1_000_000, 100_000, 8, 10), name="combine_u8_100k_8x10"),
        # index construction: lists of 64 into rows of 32, and lists of 128 into rows of 64
        dict(_build(1_000_000, 500, 64, 32), name="build_1m_64_32"),
        dict(_build(250_000, 125, 128, 64), name="build_250k_128_64"),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case of the same ranges; sizes over their logarithm, odd ones among them, below the largest listed cost."""
    kind = rng.choices(("search", "route", "combine", "build"), (6, 2, 1, 2))[0]
    dtype = rng.choice(("u8", "u8", "f16", "f32"))
    unit = 16 // SIZES[dtype]
    if kind == "search":
        dim = rng.choice({"u8": (128, 128, 96, 144, 256), "f16": (768, 128, 200, 384), "f32": (96, 128, 100, 256)}[dtype])
        mean = _log(rng, 300, 2000)
        n = min(_log(rng, 10_000, 1_000_000), 400_000_000 // (dim * SIZES[dtype]), (1 << 30) // mean)
        n = max(n, 4 * mean)
        degree = rng.choice((16, 24, 27, 32, 32, 33, 48, 64, 64))
        width = rng.choice([w for w in (1, 2, 3, 4, 4, 6, 8) if w * degree <= 512])
        itopk = rng.choice((32, 64, 100, 112, 128, 160, 184, 192, 256))
        clusters = max(4, n // mean)
        entry = rng.choice(("routed", "routed", "routed", "uniform"))
        # a query costs about list size x degree x row: no more than a quarter of the largest listed case
        most = 131_072 * (184 * 32 * 256) // (itopk * degree * (128 + dim * SIZES[dtype]))
        return _search(dtype, dim, n, clusters, degree, _log(rng, 50, max(50, min(60_000, most // 2))), min(itopk, rng.choice((1, 7, 10, 10, 32, 100))),
                       itopk, width, 200, metric=rng.choice(("l2", "l2", "ip")) if dtype != "u8" else "l2", entry=entry,
                       route_c=rng.choice((1, 1, 2, 4)), n_entry=rng.choice((16, 32, 32, 64)))
    if kind == "route":
        dim = unit * max(1, _log(rng, 32, 1024 // SIZES[dtype]) // unit)
        if dtype == "u8" and rng.random() < 0.5:
            dim = 128
        clusters = _log(rng, 100, 16_384)
        cost = clusters * dim * ({"u8": 2, "f16": 8, "f32": 40}[dtype] if dim * SIZES[dtype] % 32 == 0 else 200)
        nq = _log(rng, 100, max(100, min(500_000, int(2.0e12 / cost))))
        return _route(dtype, dim, clusters, nq, rng.choice((1, 1, 2, 4, 8)), metric=rng.choice(("l2", "ip")))
    if kind == "combine":
        dim = unit * max(1, _log(rng, 32, 1024) // unit)
        k = rng.choice((1, 7, 10, 10, 32, 100))
        parts = rng.choice([p for p in (2, 3, 4, 8) if p * k <= 512])
        nq = _log(rng, 100, min(200_000, 500_000_000 // (k * dim * SIZES[dtype])))
        return _combine(dtype, dim, _log(rng, 10_000, min(1_000_000, 500_000_000 // (dim * SIZES[dtype]))), nq, parts, k)
    d_in = rng.choice((32, 48, 64, 64, 90, 96, 128))
    d_out = min(64, rng.choice((d_in // 2, d_in // 2, d_in // 3, d_in)))
    n = _log(rng, 5_000, min(1_000_000, 250_000 * 128 * 128 // (d_in * d_in)))
    return _build(n, max(1, n // _log(rng, 500, 2000)), d_in, d_out)


# ------------------------------------------------------------------------------------------------ inputs


def _index(case, seed, device):
    """Vectors of a Gaussian mixture stored cluster by cluster, as the benchmark generates them."""
    if case["dtype"] == "u8":
        return inputs.sift_like(case["n"], case["clusters"], dim=case["dim"], seed=seed, device=device)
    return inputs.unit_mixture(case["n"], case["clusters"], case["dim"], DTYPES[case["dtype"]], METRICS[case["metric"]],
                               seed=seed, device=device)


def _queries(part, case, seed):
    make = inputs.sift_like_queries if case["dtype"] == "u8" else inputs.unit_mixture_queries
    return make(part, case["nq"], seed=seed)


def _knn(part, degree, block=1 << 28):
    """Exact nearest neighbours of every vector among its own cluster's, ascending, many clusters at a time; -1 pads."""
    x, off = part.vectors, part.offsets
    n = x.shape[0]
    graph = torch.full((n, degree), -1, dtype=torch.int32, device=x.device)
    first, size = off[:-1], off[1:] - off[:-1]
    s = int(size.max())
    step = max(1, block // (s * s))
    at = torch.arange(s, device=x.device)
    for c in range(0, size.numel(), step):
        ids = first[c:c + step].unsqueeze(1) + at
        there = at < size[c:c + step].unsqueeze(1)
        y = x[ids.clamp(max=n - 1)].float()
        key = torch.bmm(y, y.transpose(1, 2).contiguous())
        if part.metric == ann.ANN_IP:
            key.neg_()
        else:
            yy = (y * y).sum(2)
            key.mul_(-2.0).add_(yy.unsqueeze(1)).add_(yy.unsqueeze(2))
        key.masked_fill_(~there.unsqueeze(1), float("inf"))
        key.diagonal(dim1=1, dim2=2).fill_(float("inf"))
        val, col = torch.topk(key, min(degree, s), dim=2, largest=False, sorted=True)
        got = torch.where(torch.isinf(val), torch.full_like(col, -1), col + first[c:c + step].view(-1, 1, 1))
        graph[ids[there], :got.shape[2]] = got[there].to(torch.int32)
    return graph


def _graph(part, case, seed):
    """The kNN graph; where entries are drawn over the whole index, a quarter of every row are links to anywhere."""
    graph = _knn(part, case["degree"])
    if case["entry"] == "uniform":
        g = torch.Generator(device=graph.device).manual_seed(seed + 2)
        far = case["degree"] // 4
        graph[:, -far:] = torch.randint(0, case["n"], (case["n"], far), generator=g, device=graph.device, dtype=torch.int32)
    return graph


def _candidates(case, seed, device):
    """`parts` ascending lists of k candidates per query, as the partitions return them; ids of a query are distinct."""
    g = torch.Generator(device=device).manual_seed(seed)
    nq, parts, k = case["nq"], case["parts"], case["k"]
    per = case["n"] // parts
    first = torch.randint(0, per, (nq, parts, 1), generator=g, device=device)
    ids = (first + 7 * torch.arange(k, device=device)) % per * parts + torch.arange(parts, device=device).view(1, -1, 1)
    if case["dtype"] == "u8":
        keys = torch.randint(40_000, 60_000, (nq, parts, k), generator=g, device=device, dtype=torch.int32)
    else:
        keys = torch.rand((nq, parts, k), generator=g, device=device) * 0.2 + 0.15
    keys = torch.sort(keys, dim=2).values
    return ids.to(torch.int32).view(nq, -1).contiguous(), keys.view(nq, -1).contiguous()


def _table(case, seed, device):
    g = torch.Generator(device=device).manual_seed(seed + 1)
    if case["dtype"] == "u8":
        return torch.randint(0, 256, (case["n"], case["dim"]), generator=g, device=device, dtype=torch.uint8)
    return (torch.randn((case["n"], case["dim"]), generator=g, device=device) / case["dim"] ** 0.5).to(DTYPES[case["dtype"]])


def _centroids(case, seed, device):
    """Centroids and queries of a mixture; no vectors are needed for the routing."""
    few = dict(case, n=case["clusters"])
    part = _index(few, seed, device)
    return part, _queries(part, case, seed + 1)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "build":
        part = inputs.sift_like(case["n"], case["clusters"], seed=seed, device=DEVICE)
        knn = _knn(part, case["d_in"])
        need = ann.ann_graph_optimize_workspace_bytes(case["n"], case["d_in"], case["d_out"])
        return dict(kind=kind, knn=knn, d_out=case["d_out"], workspace=torch.empty(need, dtype=torch.uint8, device=DEVICE))
    if kind == "combine":
        ids, keys = _candidates(case, seed, DEVICE)
        table = _table(case, seed, DEVICE)
        graph = torch.full((case["n"], 1), -1, dtype=torch.int32, device=DEVICE)  # the table is only read from
        return dict(kind=kind, ids=ids, keys=keys, k=case["k"], handle=ann.ann_index_load(table, graph))
    if kind == "route":
        part, queries = _centroids(case, seed, DEVICE)
        graph = torch.full((case["clusters"], 1), -1, dtype=torch.int32, device=DEVICE)
        h = ann.ann_index_load(part.vectors, graph, metric=METRICS[case["metric"]], entry_mode=ann.ANN_ENTRY_ROUTED,
                               centroids=part.centres, cluster_offsets=part.offsets, route_c=case["route_c"])
        return dict(kind=kind, handle=h, queries=queries)
    part = _index(case, seed, DEVICE)
    routed = dict(entry_mode=ann.ANN_ENTRY_ROUTED, centroids=part.centres, cluster_offsets=part.offsets, route_c=case["route_c"])
    h = ann.ann_index_load(part.vectors, _graph(part, case, seed), metric=METRICS[case["metric"]], n_entry=case["n_entry"],
                           seed=seed + 3, **(routed if case["entry"] == "routed" else {}))
    return dict(kind=kind, handle=h, queries=_queries(part, case, seed + 1),
                how=(case["k"], case["itopk"], case["width"], case["iters"]))


def run(state):
    kind = state["kind"]
    if kind == "search":
        return ann.ann_search(state["handle"], state["queries"], *state["how"])
    if kind == "route":
        return ann.ann_route(state["handle"], state["queries"])
    if kind == "combine":
        ids, keys = ann.ann_merge_topk(state["ids"], state["keys"], state["k"])
        return ids, keys, ann.ann_gather_vectors(state["handle"], ids)
    return ann.ann_graph_optimize(state["knn"], state["d_out"], workspace=state["workspace"])


# ------------------------------------------------------------------------------------------------ what a pass cannot do without


def work(case):
    kind = case["kind"]
    if kind == "build":
        # the lists are read once and the rows written once; an edge x -> y of rank j is looked for in j rows
        n, d_in, d_out = case["n"], case["d_in"], case["d_out"]
        return {"bytes": n * (d_in + d_out) * 4, "flops": n * d_in * d_in}
    row = case["dim"] * SIZES[case["dtype"]]
    if kind == "combine":
        cand, out = case["nq"] * case["parts"] * case["k"], case["nq"] * case["k"]
        return {"bytes": cand * 8 + out * 8 + min(out, case["n"]) * row + out * row, "flops": cand}
    if kind == "route":
        return {"bytes": (case["nq"] + case["clusters"]) * row + case["nq"] * case["route_c"] * 4,
                "flops": 2 * case["nq"] * case["clusters"] * case["dim"]}
    # a search that runs to its end expands about every entry of its list; a parent gives up to eight new rows, fewer
    # where its cluster is used up
    mean = case["n"] / case["clusters"]
    parents = min(case["itopk"], case["width"] * case["iters"])
    rows = min(parents * min(8, case["degree"]), mean * (case["route_c"] if case["entry"] == "routed" else 4)) + case["n_entry"]
    nq = case["nq"]
    read = min(nq * rows, case["n"]) * row + min(nq * parents, case["n"]) * case["degree"] * 4
    flops = nq * rows * case["dim"] * (3 if case["metric"] == "l2" else 2)
    if case["entry"] == "routed":
        read += case["clusters"] * row
        flops += 2 * nq * case["clusters"] * case["dim"]
    return {"bytes": read + nq * (row + case["k"] * 8), "flops": flops}


def tolerance(case):
    if case["kind"] in ("build", "combine") or case["dtype"] == "u8":
        return "exact"
    if case["kind"] == "route":
        # centroids whose keys differ by less than the sums' rounding may change places: none of 500 000 did against 64 bits
        return {"rel": 0.0, "differ": 0.0005}
    # keys are 32-bit sums, at most 5e-8 (all) and 2e-7 (one) off 64 bits; neighbours whose keys differ by less than that
    # may change places: up to 6e-4 of the ids of an inner-product index do against 64 bits
    return {"rel": 2e-7, "max": 1e-6, "differ": 0.0025}


# ------------------------------------------------------------------------------------------------ the same in 64 bits


def _shift(z, bits):
    return (z >> bits) & ((1 << (64 - bits)) - 1)


def _wrap(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _splitmix_mod(seed, counter, modulus):
    """(output `counter` of the splitmix64 stream) mod `modulus`, in wrapping int64 arithmetic."""
    z = _wrap(seed) + (counter + 1) * _wrap(0x9E3779B97F4A7C15)
    z = (z ^ _shift(z, 30)) * _wrap(0xBF58476D1CE4E5B9)
    z = (z ^ _shift(z, 27)) * _wrap(0x94D049BB133111EB)
    z = z ^ _shift(z, 31)
    return (_shift(z, 1) % modulus * 2 + (z & 1)) % modulus


def _keys(q, rows, metric):
    """Keys of rows [b, m, dim] against q [b, dim], in 64 bits."""
    if metric == "ip":
        return -torch.matmul(rows.double(), q.double().unsqueeze(2)).squeeze(2)
    return (rows.double() - q.double().unsqueeze(1)).square_().sum(2)


def _routes(queries, centres, metric, c):
    """The c nearest centroids under (key, index); ascending."""
    got = []
    y = centres.double()
    step = max(1, (1 << 27) // centres.shape[0])
    for lo in range(0, queries.shape[0], step):
        x = queries[lo:lo + step].double()
        key = x @ y.T
        key = key.neg_() if metric == "ip" else key.mul_(-2.0).add_((y * y).sum(1))
        if c == 1:
            got.append(torch.argmin(key, 1, keepdim=True) if queries.dtype != torch.uint8 else
                       (key == key.amin(1, keepdim=True)).to(torch.uint8).argmax(1, keepdim=True))
        else:
            got.append(torch.sort(key, dim=1, stable=True).indices[:, :c])
    return torch.cat(got)


_NONE = (1 << 31) - 1


def _by_key_then_id(key, ids, *more):
    o = torch.argsort(ids, dim=1, stable=True)
    o = torch.gather(o, 1, torch.argsort(torch.gather(key, 1, o), dim=1, stable=True))
    return [torch.gather(t, 1, o) for t in (key, ids, *more)]


def _beam_search(case, part, graph, queries, first, seed):
    """ids, keys of queries number first, first + 1, ...: the documented search, many queries side by side."""
    b, dev = queries.shape[0], queries.device
    k, itopk, width = case["k"], case["itopk"], case["width"]
    at = (first + torch.arange(b, device=dev)).unsqueeze(1) * case["n_entry"] + torch.arange(case["n_entry"], device=dev)
    if case["entry"] == "uniform":
        cand = _splitmix_mod(seed + 3, at, torch.full_like(at, case["n"]))
    else:
        c = _routes(queries, part.centres, case["metric"], case["route_c"])
        c = c[:, torch.arange(case["n_entry"], device=dev) % case["route_c"]]
        lo, size = part.offsets[c], part.offsets[c + 1] - part.offsets[c]
        cand = torch.where(size > 0, lo + _splitmix_mod(seed + 3, at, size.clamp(min=1)), torch.full_like(lo, _NONE))
    ids = torch.full((b, itopk), _NONE, dtype=torch.int64, device=dev)
    key = torch.full((b, itopk), float("inf"), dtype=torch.float64, device=dev)
    done = torch.ones((b, itopk), dtype=torch.bool, device=dev)
    for rnd in range(case["iters"] + 1):
        # drop what the list holds already and what stands twice; anything else scored before is rejected again by its key
        cand = torch.sort(cand, dim=1).values
        cand[:, 1:][cand[:, 1:] == cand[:, :-1]] = _NONE
        held = torch.sort(ids, dim=1).values.contiguous()
        pos = torch.searchsorted(held, cand).clamp_(max=itopk - 1)
        cand = torch.where(torch.gather(held, 1, pos) == cand, torch.full_like(cand, _NONE), cand)
        new = torch.full(cand.shape, float("inf"), dtype=torch.float64, device=dev)
        step = max(1, (1 << 27) // (cand.shape[1] * case["dim"]))
        for r in range(0, b, step):
            new[r:r + step] = _keys(queries[r:r + step], part.vectors[cand[r:r + step].clamp(max=case["n"] - 1)], case["metric"])
        new[cand == _NONE] = float("inf")
        key, ids, done = _by_key_then_id(torch.cat([key, new], 1), torch.cat([ids, cand], 1),
                                         torch.cat([done, cand == _NONE], 1))
        key, ids, done = key[:, :itopk], ids[:, :itopk], done[:, :itopk]
        open_ = ~done
        take = open_ & (open_.cumsum(1) <= width)
        if rnd == case["iters"] or not bool(take.any()):
            break
        slot = torch.where(take, take.cumsum(1) - 1, torch.full_like(ids, width))
        parent = torch.full((b, width + 1), -1, dtype=torch.int64, device=dev).scatter_(1, slot, ids)[:, :width]
        done = done | take
        cand = graph[parent.clamp(min=0)].long()
        cand[(parent < 0) | (parent >= case["n"])] = -1
        cand = cand.view(b, -1)
        cand[(cand < 0) | (cand >= case["n"])] = _NONE
    ids, key = ids[:, :k], key[:, :k]
    return torch.where(ids == _NONE, torch.full_like(ids, -1), ids).to(torch.int32), key


def exact(case, seed, device=DEVICE):
    kind = case["kind"]
    if kind == "build":
        return None  # whole numbers throughout: there is nothing to round
    if kind == "route":
        part, queries = _centroids(case, seed, device)
        if case["nq"] * case["clusters"] > 4e9:
            return None
        return _routes(queries, part.centres, case["metric"], case["route_c"]).to(torch.int32)
    if kind == "combine":
        ids, keys = _candidates(case, seed, device)
        key, ids = _by_key_then_id(keys.double(), ids)
        ids, key = ids[:, :case["k"]], key[:, :case["k"]]
        return ids, key.to(torch.int32) if case["dtype"] == "u8" else key, _table(case, seed, device)[ids.long()]
    if case["nq"] * case["itopk"] * case["degree"] * case["dim"] > 1e11:
        return None  # minutes
    part = _index(case, seed, device)
    graph = _graph(part, case, seed)
    queries = _queries(part, case, seed + 1)
    step = 4096
    got = [_beam_search(case, part, graph, queries[lo:lo + step], lo, seed) for lo in range(0, case["nq"], step)]
    ids, key = (torch.cat(v) for v in zip(*got))
    return ids, key.to(torch.int32) if case["dtype"] == "u8" else key
