"""The work that a user of this library has it do, as cases that can be timed.

A case is a dict of plain values; `prepare` makes on the GPU what a training program holds
before it asks for a mini-batch (the graph handle over its CSC arrays, the feature tables,
the shuffled seeds, the pipeline), and `run` makes one pass through the public entry points.

Graphs ("graph", scaled in nodes and edges by "scale"):
  tiny      two node types, three edge types, 100k edges (the smallest calls)
  academic  paper / author / institution / field, 4 relations and their reverses, 42M edges
  share     user / item / seller, 3 relations and their reverses, 1.2G edges: one GPU's share of
            a billion-edge graph, with hubs of millions of in-edges
  kg        one node type, "relations" relations of Zipf(1.2) sizes, 300M edges on 20M entities
In-degrees follow a discrete power law (pmf ~ k^-alpha), sources are uniform; a reverse type is
the transpose of its forward type.

Paths ("path"):
  sample    vertex-seeded mini-batches with their input features: one call, or a bundle
  pipeline  the same through worker streams, in bundles, returned in order
  link      edge-seeded mini-batches: one negative per target, targets and reverses excluded
  layers    layer-wise (LADIES) mini-batches, "draws" vertices per node type and hop
  rows      a pull of feature rows by vertex ID

Every output is an integer or a copied feature row, so outputs are compared exactly.

The sizes of a mini-batch follow from its vertices and the graph, and a case's outputs keep their
shapes from seed to seed: the adjacency and the members of each batch are made from the case's
own values, while the seed makes the features, the order of each batch (and with it the order of
every block array and local ID) and, for a row pull, the IDs.
"""
import json
import math
import zlib

import numpy as np
import torch

import paper_2112_15345_amd as hg

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}

# alpha, node types (count, featured), forward edge types (source, destination, edges), reverses
GRAPHS = {
    "tiny": (1.5, ((6_000, True), (4_000, True)),
             ((0, 0, 40_000), (0, 1, 30_000), (1, 0, 30_000)), False),
    "academic": (2.1, ((736_000, True), (1_130_000, True), (8_700, True), (60_000, True)),
                 ((1, 0, 7_100_000), (0, 0, 5_400_000), (0, 3, 7_500_000), (1, 2, 1_000_000)),
                 True),
    "share": (1.8, ((60_000_000, True), (30_000_000, True), (2_000_000, False)),
              ((0, 1, 450_000_000), (0, 0, 120_000_000), (1, 2, 30_000_000)), True),
    "kg": (2.1, ((20_000_000, True),), None, False),
}
KG_EDGES = 300_000_000
SEED_TYPE = 0     # papers, users, entities, the tiny graph's first type
LINK_ETYPE = 1    # link prediction's targets: paper cites paper


def listed():
    return [
        # an interactive or debugging call: 64 seeds on a small graph, every block array read;
        # launches and waits are all there is
        {"name": "tiny batch", "path": "sample", "graph": "tiny", "scale": 1.0, "dtype": "f32",
         "dim": 16, "fanout": "5,5", "batch": 64, "bundle": 1, "out": "blocks"},
        # one training mini-batch at the usual batch size, asked for when it is needed
        {"name": "academic batch", "path": "sample", "graph": "academic", "scale": 1.0,
         "dtype": "f32", "dim": 128, "fanout": "25,20", "batch": 1024, "bundle": 1,
         "out": "inputs"},
        # the same made ahead in a bundle, the throughput of training
        {"name": "academic bundle", "path": "sample", "graph": "academic", "scale": 1.0,
         "dtype": "f32", "dim": 128, "fanout": "25,20", "batch": 1024, "bundle": 16,
         "out": "features"},
        # wide 16-bit features and large batches: the feature copy dominates
        {"name": "wide features", "path": "sample", "graph": "academic", "scale": 1.0,
         "dtype": "bf16", "dim": 512, "fanout": "10,10", "batch": 8192, "bundle": 8,
         "out": "inputs"},
        # offline inference over a node type: every in-edge of a large block of seeds, rows of
        # 200 bytes (no multiple of 16)
        {"name": "full neighbours", "path": "sample", "graph": "academic", "scale": 1.0,
         "dtype": "f16", "dim": 100, "fanout": "-1", "batch": 50_001, "bundle": 1,
         "out": "inputs"},
        # many relations, nearly every (vertex, relation) pair empty
        {"name": "knowledge graph", "path": "sample", "graph": "kg", "scale": 1.0,
         "relations": 200, "dtype": "f32", "dim": 64, "fanout": "10,10", "batch": 2048,
         "bundle": 4, "out": "inputs"},
        # one mini-batch of the billion-edge share: hubs of millions of in-edges
        {"name": "share batch", "path": "sample", "graph": "share", "scale": 1.0, "dtype": "f16",
         "dim": 128, "fanout": "15,10,5", "batch": 4096, "bundle": 1, "out": "inputs"},
        # the same as a trainer has it made ahead: three worker streams, bundles of two
        {"name": "share pipeline", "path": "pipeline", "graph": "share", "scale": 1.0,
         "dtype": "f16", "dim": 128, "fanout": "15,10,5", "batch": 4096, "bundle": 2, "units": 6,
         "workers": 3, "out": "inputs"},
        # link prediction: 1000 citations and as many negatives, reverse edges left out
        {"name": "link prediction", "path": "link", "graph": "academic", "scale": 1.0,
         "dtype": "f32", "dim": 128, "fanout": "25,15", "batch": 1000, "bundle": 8,
         "out": "features"},
        # layer-wise sampling, 512 vertices per node type in each of two hops
        {"name": "layer-wise", "path": "layers", "graph": "academic", "scale": 1.0,
         "dtype": "f32", "dim": 128, "draws": 512, "hops": 2, "batch": 1024, "bundle": 16,
         "out": "features"},
        # features kept in host memory (pinned), pulled over the host link
        {"name": "host features", "path": "sample", "graph": "academic", "scale": 0.25,
         "dtype": "f32", "dim": 128, "fanout": "25,20", "batch": 1024, "bundle": 4,
         "host": True, "out": "features"},
        # a row pull of an odd number of odd-sized rows (evaluation, caching)
        {"name": "row pull", "path": "rows", "nodes": 1_130_001, "dtype": "f32", "dim": 100,
         "rows": 200_003},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["sample"] * 6 + ["pipeline", "link", "layers", "rows"])
    dtype = rng.choice(["f32", "f16", "bf16"])
    dim = rng.choice([16, 64, 100, 128, 256, 33])
    if path == "rows":
        return {"path": "rows", "nodes": _log_int(rng, 10_000, 4_000_000), "dtype": dtype,
                "dim": rng.choice([33, 64, 100, 128, 512, 768]),
                "rows": _log_int(rng, 64, 400_000)}
    graph = rng.choice({"sample": ["tiny", "academic", "academic", "share", "kg"],
                        "pipeline": ["academic", "share"]}.get(path, ["academic"]))
    case = {"path": path, "graph": graph, "dtype": dtype, "dim": dim}
    if graph == "tiny":
        case["scale"] = round(math.exp(rng.uniform(0, math.log(8))), 3)
        case["batch"], case["bundle"] = _log_int(rng, 16, 1500), rng.choice([1, 1, 2])
        case["fanout"] = rng.choice(["5,5", "10,10", "3,3,3", "15"])
    elif graph == "academic":
        case["scale"] = round(math.exp(rng.uniform(math.log(1 / 16), 0)), 3)
        case["batch"] = _log_int(rng, 100, 4000)
        case["bundle"] = rng.choice([1, 1, 2, 5, 8, 13, 16])
        case["fanout"] = rng.choice(["25,20", "25,15", "10,10", "15,10,5", "-1", "20"])
    elif graph == "share":
        case["scale"] = round(math.exp(rng.uniform(math.log(1 / 16), 0)), 3)
        case["batch"] = _log_int(rng, 500, 4096)
        case["bundle"] = rng.choice([1, 1, 2, 3])
        case["fanout"] = rng.choice(["15,10,5", "15,10", "10,10"])
        case["dtype"], case["dim"] = rng.choice(["f16", "bf16"]), min(dim, 128)
    else:
        case["dim"] = min(dim, 128)
        case["scale"] = round(math.exp(rng.uniform(math.log(1 / 16), 0)), 3)
        case["relations"] = _log_int(rng, 20, 200)
        case["batch"] = _log_int(rng, 200, 2048)
        case["bundle"] = rng.choice([1, 2, 4])
        case["fanout"] = rng.choice(["10,10", "15", "20,5"])
    if path == "pipeline":
        case["workers"] = rng.choice([2, 3])
        case["bundle"] = rng.choice([1, 2])
        case["units"] = rng.choice([3, 4, 6])
    if path == "link":
        case["fanout"] = rng.choice(["25,15", "10,10"])
        case["bundle"] = rng.choice([1, 3, 8])
    if path == "layers":
        del case["fanout"]
        case["draws"], case["hops"] = rng.choice([64, 256, 512]), 2
    case["out"] = "features"
    if path == "sample" and case["bundle"] == 1:
        case["out"] = "blocks" if graph == "tiny" else "inputs"
    while work(case)["bytes"] > 1e10:  # no more than the largest listed case
        case["batch"] //= 2
    return case


# ---- the graph ---------------------------------------------------------------------------


def _types(case):
    """alpha, node types [(count, featured)], edge types [(source, destination, edges, forward
    type of a reverse or None)]."""
    alpha, nts, ets, reverse = GRAPHS[case["graph"]]
    s = case["scale"]
    nts = [(max(int(n * s), 64), f) for n, f in nts]
    if ets is None:
        R = case["relations"]
        w = [(r + 1) ** -1.2 for r in range(R)]
        ets = [(0, 0, KG_EDGES * x / sum(w)) for x in w]
    ets = [(a, b, max(int(n * s), 1)) for a, b, n in ets]
    out = [(a, b, n, None) for a, b, n in ets]
    if reverse:
        out += [(b, a, n, e) for e, (a, b, n) in enumerate(ets)]
    return alpha, nts, out


def _degrees(n_dst, n_src, edges, alpha, gen):
    u = 1.0 - torch.rand(n_dst, generator=gen, device="cuda", dtype=torch.float64)
    raw = torch.floor(u.pow_(-1.0 / (alpha - 1.0))).clamp_(max=float(n_src))
    x = raw.mul_(edges / raw.sum())
    d = torch.floor(x)
    d += torch.rand(n_dst, generator=gen, device="cuda", dtype=torch.float64) < (x - d)
    return d.clamp_(max=float(n_src)).to(torch.int64)


def _indptr(deg):
    ip = torch.zeros(deg.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(deg, 0, out=ip[1:])
    return ip


def _edges(case, gen):
    """CSC (source type, destination type, indptr, indices) of every edge type, and the reverse
    maps (edge type, edge IDs) of link prediction."""
    alpha, nts, ets = _types(case)
    want_maps = case["path"] == "link"
    built, maps = [], {}
    for s, d, n, fwd in ets:
        if fwd is None:
            deg = _degrees(nts[d][0], nts[s][0], n, alpha, gen)
            ip = _indptr(deg)
            ix = torch.randint(nts[s][0], (int(ip[-1]),), generator=gen, device="cuda",
                               dtype=torch.int64)
            built.append((s, d, ip, ix))
            continue
        # the transpose: slots ordered by (source, destination) of the forward type
        _, _, ip, ix = built[fwd]
        n_d = nts[s][0]
        dst = torch.repeat_interleave(torch.arange(n_d, device="cuda"), ip[1:] - ip[:-1])
        key = ix * n_d + dst
        del dst
        key, order = torch.sort(key, stable=True) if want_maps else (torch.sort(key)[0], None)
        rip = _indptr(torch.bincount(ix, minlength=nts[d][0]))
        built.append((s, d, rip, key.remainder_(n_d)))
        if want_maps:
            fmap = torch.empty_like(order)
            fmap[order] = torch.arange(order.numel(), device="cuda")
            maps[fwd], maps[len(built) - 1] = (len(built) - 1, fmap), (fwd, order)
    return built, maps


def _features(n, case, gen):
    x = torch.empty((n, case["dim"]), dtype=DTYPES[case["dtype"]], device="cuda")
    for r in range(0, n, 1 << 22):
        x[r:r + (1 << 22)].normal_(generator=gen)
    if case.get("host"):
        x = torch.empty(x.shape, dtype=x.dtype, pin_memory=True).copy_(x)
    return x


def _fanouts(case, R):
    return [[int(k)] * R for k in case["fanout"].split(",")]


def _structure_seed(case):
    """The same for every case over the same values: its name and the outputs read are left out."""
    values = {k: v for k, v in case.items() if k not in ("name", "out")}
    return zlib.crc32(json.dumps(values, sort_keys=True).encode())


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["path"] == "rows":
        table = _features(case["nodes"], case, gen)
        ids = torch.randint(case["nodes"], (case["rows"],), generator=gen, device="cuda")
        return {"graph": hg.Graph([(case["nodes"], table)], []), "ids": ids, "case": case}
    _, nts, _ = _types(case)
    same = torch.Generator(device="cuda")
    same.manual_seed(_structure_seed(case))
    ets, maps = _edges(case, same)
    feats = [_features(n, case, gen) if f else None for n, f in nts]
    g = hg.Graph([(n, f) for (n, _), f in zip(nts, feats)], ets)
    T, R = len(nts), len(ets)
    st = {"graph": g, "case": case}
    total = case["bundle"] * case.get("units", 1)
    if case["path"] == "link":
        pool = int(ets[LINK_ETYPE][3].numel())
    else:
        pool = nts[SEED_TYPE][0]
    # an epoch's shuffle, cut into batches
    batch = max(1, min(case["batch"], pool // total))
    picks = torch.randperm(pool, generator=same, device="cuda")[:batch * total]
    at = LINK_ETYPE if case["path"] == "link" else SEED_TYPE
    st["seeds"] = []
    for b in range(total):
        row = [None] * (R if case["path"] == "link" else T)
        order = torch.randperm(batch, generator=gen, device="cuda")
        row[at] = picks[b * batch:(b + 1) * batch][order]
        st["seeds"].append(row)
    st["rng"] = [_structure_seed(case) * 1000003 + b for b in range(total)]
    if case["path"] == "layers":
        st["sizes"] = [[case["draws"]] * T for _ in range(case["hops"])]
    else:
        st["fanouts"] = _fanouts(case, R)
    if case["path"] == "link":
        st["rev_etype"] = [maps[e][0] for e in range(R)]
        st["rev_eid"] = [maps[e][1] for e in range(R)]
    if case["path"] == "pipeline":
        st["pipe"] = hg.Pipeline(g, workers=case["workers"], capacity=total)
    return st


# ---- one pass ----------------------------------------------------------------------------


def _outputs(case, g, batches):
    """What a program reads of each mini-batch: its input features, then (as far as the number
    of arrays allows) its input vertices, or every array of every block."""
    out = []
    for b in batches:
        out.append([b.features(t) for t in range(g.T) if g.ntypes[t][1] is not None])
        if case["path"] == "link":
            out.append(list(b.edge_pairs(LINK_ETYPE)))
        if case["out"] == "inputs":
            out.append([b.input_nodes(t) for t in range(g.T)])
        elif case["out"] == "blocks":
            out.append([b.nodes(h, t)[1] for h in range(b.n_hops) for t in range(g.T)])
            out.append([list(b.edges(h, e)) for h in range(b.n_hops) for e in range(g.R)])
    return out


def run(state):
    g, case = state["graph"], state["case"]
    if case["path"] == "rows":
        return g.gather_rows(0, state["ids"])
    seeds, rng = state["seeds"], state["rng"]
    if case["path"] == "pipeline":
        pipe, k = state["pipe"], case["bundle"]
        for u in range(case["units"]):
            pipe.submit_bundle(seeds[u * k:(u + 1) * k], state["fanouts"], rng[u * k:(u + 1) * k])
        got = [pipe.next() for _ in range(len(seeds))]
    elif case["path"] == "link":
        got = g.sample_edge_bundle(seeds, state["fanouts"], rng, n_neg=1,
                                   exclude=hg.HG_EXCLUDE_REVERSE, rev_etype=state["rev_etype"],
                                   rev_eid=state["rev_eid"], gather="all")
    elif case["path"] == "layers":
        got = g.sample_layers_bundle(seeds, state["sizes"], rng, gather="all")
    elif len(seeds) == 1:
        got = [g.sample_blocks(seeds[0], state["fanouts"], rng[0], gather="all")]
    else:
        got = g.sample_bundle(seeds, state["fanouts"], rng, gather="all")
    return _outputs(case, g, got)


# ---- what a pass cannot do without ---------------------------------------------------------


def _degree_grid(n_dst, n_src, edges, alpha):
    """In-degrees at some 3000 quantiles (weights sum to n_dst), by the generator's power law."""
    edges_u = np.concatenate([np.logspace(-math.log10(max(n_dst, 10)), -2, 1500),
                              np.linspace(0.01, 1, 1500)[1:]])
    u = 0.5 * (edges_u[1:] + edges_u[:-1])
    w = np.diff(edges_u) * n_dst
    raw = np.minimum(np.floor(u ** (-1.0 / (alpha - 1.0))), n_src)
    return raw * (edges / (raw * w).sum()), w


def _kept(d, w, K, n):
    """Mean over vertices weighted by w of the kept in-edges (fractional degrees are rounded
    at random by the generator) and of the keyed ones."""
    lo = np.floor(d)
    f = d - lo
    cap = (lambda x: np.minimum(x, K)) if K >= 0 else (lambda x: x)
    kept = (1 - f) * cap(lo) + f * cap(lo + 1)
    keyed = np.where(d > K, d, 0.0) if K >= 0 else 0 * d
    return (kept * w).sum() / n, (keyed * w).sum() / n


def work(case):
    """Bytes: the frontier and its in-edge ranges read, the kept edges' sources read, the block
    arrays written, the input rows read and written.  Operations: 37 integer operations per
    four random keys, one key for every in-edge of a pair that selects (the result is defined
    by them).  Sizes are expectations over the generator's degree law."""
    size = torch.empty(0, dtype=DTYPES[case["dtype"]]).element_size()
    row = size * case["dim"]
    if case["path"] == "rows":
        return {"bytes": float(case["rows"] * (8 + 2 * row)), "flops": 0.0}
    alpha, nts, ets = _types(case)
    layers = case["path"] == "layers"
    total = case["bundle"] * case.get("units", 1)
    batch = case["batch"]
    # the frontier of each type in parts: [count, forward type whose in-degree biases it, the
    # inclusion weights of that type's quantiles]
    parts = [[] for _ in nts]
    grids = {}
    for e, (s, d, n, fwd) in enumerate(ets):
        if fwd is None:
            grids[e] = _degree_grid(nts[d][0], nts[s][0], n, alpha)
    if case["path"] == "link":
        s, d, _, _ = ets[LINK_ETYPE]
        x, w = grids[LINK_ETYPE]
        parts[s].append([batch, None, None])
        parts[d] += [[batch, LINK_ETYPE, w * x], [batch, None, None]]
    else:
        parts[SEED_TYPE].append([min(batch, nts[SEED_TYPE][0]), None, None])
    fan = [-1] * case["hops"] if layers else [int(k) for k in case["fanout"].split(",")]
    nbytes, ops = 0.0, 0.0
    for K in fan:
        front = [sum(q[0] for q in p) for p in parts]
        got = [[] for _ in nts]
        for e, (s, d, n, fwd) in enumerate(ets):
            kept = keyed = 0.0
            for c, bias, incl in parts[d]:
                if fwd is not None:  # near-Poisson in-degrees: the mean, cut at K
                    m = n / nts[d][0]
                    k1 = m if K < 0 else min(m, K)
                    q1 = m if 0 <= K < m else 0.0
                elif bias == e:
                    k1, q1 = _kept(grids[e][0], incl, K, max(incl.sum(), 1e-9))
                else:
                    k1, q1 = _kept(grids[e][0], grids[e][1], K, nts[d][0])
                kept += c * k1
                keyed += c * q1
            kept = min(kept, float(n))
            nbytes += 16 * front[d] + 8 * front[d]     # in-edge ranges, block CSC
            if layers:
                nbytes += 8 * kept                     # every in-edge's source
            else:
                nbytes += (8 + 16) * kept              # source read; edge and local IDs written
                ops += 37 / 4 * keyed
            # distinct sources: uniform, or by the forward type's in-degree
            if fwd is None:
                got[s].append([nts[s][0] * -math.expm1(-kept / nts[s][0]), None, None])
            else:
                x, w = grids[fwd]
                p = x / (x * w).sum()
                incl = w * -np.expm1(-kept * p)
                got[s].append([float(incl.sum()), fwd, incl])
        for t, (n, _) in enumerate(nts):
            if layers:
                drawn = min(float(case["draws"]), sum(p[0] for p in got[t]))
                parts[t] = parts[t] + [[drawn, None, None]]
            else:
                parts[t] = parts[t] + got[t]
            c = sum(p[0] for p in parts[t])
            if c > n:
                parts[t] = [[p[0] * n / c, p[1], p[2]] for p in parts[t]]
            nbytes += 16 * min(c, n)  # frontier read, source list written
    for t, (n, featured) in enumerate(nts):
        if featured:
            nbytes += (8 + 2 * row) * sum(p[0] for p in parts[t])
    return {"bytes": float(total * nbytes), "flops": float(total * ops)}


def tolerance(case):
    return "exact"


# ---- the same by plain numpy, for the smallest cases ---------------------------------------


def _philox(c, k0, k1):
    """Philox4x32-10 on uint64 arrays holding 32-bit words."""
    m = np.uint64(0xFFFFFFFF)
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m,
             (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _keys(eid, hop, etype, seed):
    g = eid.astype(np.uint64) >> np.uint64(2)
    c = [g & np.uint64(0xFFFFFFFF), g >> np.uint64(32), np.full_like(g, hop),
         np.full_like(g, etype)]
    r = np.stack(_philox(c, seed & 0xFFFFFFFF, seed >> 32))
    return r[(eid & 3).astype(np.int64), np.arange(eid.size)]


def exact(case, seed):
    if case["path"] == "rows":
        st = prepare(case, seed)
        return st["graph"].ntypes[0][1].double()[st["ids"]]
    if case["path"] != "sample" or case["graph"] != "tiny" or case["bundle"] != 1:
        return None
    st = prepare(case, seed)
    g = st["graph"]
    ets = [(s, d, ip.cpu().numpy(), ix.cpu().numpy()) for s, d, ip, ix in g.etypes]
    front = [np.zeros(0, np.int64) if s is None else s.cpu().numpy() for s in st["seeds"][0]]
    nodes, edges = [], []
    for h, row in enumerate(st["fanouts"]):
        kept = []
        for e, (s, d, ip, ix) in enumerate(ets):
            got = []
            for v in front[d]:
                eid = np.arange(ip[v], ip[v + 1])
                if row[e] >= 0 and eid.size > row[e]:
                    order = np.lexsort((eid, _keys(eid, h, e, st["rng"][0])))
                    eid = np.sort(eid[order[:row[e]]])
                got.append(eid)
            kept.append(got)
        new = []
        for t in range(g.T):
            src = [ets[e][3][k] for e in range(g.R) if ets[e][0] == t for k in kept[e]]
            u = np.unique(np.concatenate(src + [np.zeros(0, np.int64)]))
            new.append(np.concatenate([front[t], np.setdiff1d(u, front[t])]).astype(np.int64))
        for e, (s, d, ip, ix) in enumerate(ets):
            n = np.array([k.size for k in kept[e]], np.int64)
            eid = np.concatenate(kept[e] + [np.zeros(0, np.int64)]).astype(np.int64)
            local = np.full(g.ntypes[s][0], -1, np.int32)
            local[new[s]] = np.arange(new[s].size)
            edges.append([np.concatenate([[0], np.cumsum(n)]).astype(np.int64), local[ix[eid]],
                          np.repeat(np.arange(n.size, dtype=np.int32), n), eid])
        nodes += new
        front = new
    feats = [g.ntypes[t][1][torch.as_tensor(front[t], device="cuda")].double()
             for t in range(g.T)]
    return [feats, nodes, edges]
