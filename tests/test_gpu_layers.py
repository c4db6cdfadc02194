"""Layer-wise (LADIES) mini-batches: the HIP path through the C ABI against
the CPU oracle, element by element (every hop's source lists, every block
array, gathered bytes), on random heterographs with every kind of layer size,
on draws that land on interval boundaries, on hubs whose importance rounds to
zero, and on the academic workload's graph."""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2112_15345_amd as hg
import pins
import workloads as W
from gpu_harness import (compare, csc, frontier_in_edges, gpu_graph, gpu_seeds, internal,
                         many_relations, result_dict)

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def olib():
    return oracle.load()


def run_layer_both(olib, nn, ets, feats, seeds, sizes, sigma, g=None):
    g = g or gpu_graph(nn, ets, feats)
    featured = [t for t, f in enumerate(feats) if f is not None]
    b = g.sample_layers(gpu_seeds(seeds), sizes, sigma, gather=featured)
    got = result_dict(g, b)
    ref = oracle.HostGraph(list(zip(nn, feats)), ets, lib=olib).sample_layers(seeds, sizes, sigma)
    return g, b, ref, got


@pytest.mark.parametrize("chunk", range(3))
def test_layer_random_heterographs(olib, chunk):
    rng = np.random.default_rng(7000 + chunk)
    for c in range(40):
        nn, ets, feats, seeds, sizes, sigma = pins.random_layer_case(rng, max_nodes=60,
                                                                     max_deg=40)
        say(f"layer chunk {chunk} case {c}: T={len(nn)} R={len(ets)} sizes={sizes}")
        g, b, ref, got = run_layer_both(olib, nn, ets, feats, seeds, sizes, sigma)
        diffs = compare(ref, got, len(nn), len(ets), len(sizes))
        assert not diffs, f"case {c}: " + "\n".join(diffs[:10])
        fails = pins.check_layer_blocks(nn, ets, seeds, sizes, sigma, got)
        assert not fails, "\n".join(fails[:5])
        for t, f in enumerate(feats):
            if f is not None:
                assert b.features(t).cpu().numpy().tobytes() == f[got["input"][t]].tobytes()
        # the same graph again with other draws: the importance array and the
        # flags were left clean
        sigma2 = (sigma * 3 + 1) & (2**64 - 1)
        g, b, ref, got = run_layer_both(olib, nn, ets, feats, seeds, sizes, sigma2, g=g)
        diffs = compare(ref, got, len(nn), len(ets), len(sizes))
        assert not diffs, f"case {c} again: " + "\n".join(diffs[:10])


def test_layer_boundary_draws(olib):
    """One destination of in-degree 65536: every source has importance 1, so
    each draw r lands on the first point of candidate r's interval; the second
    hop draws among their ring neighbours."""
    n, d = 65536 + 70000, 65536
    indptr = np.concatenate([[0], d + np.arange(0, n, dtype=np.int64)])
    indices = np.concatenate([np.arange(1, d + 1), 65537 + (np.arange(1, n) % 69999)])
    ets = [(0, 0, indptr.astype(np.int64), indices.astype(np.int64))]
    g = gpu_graph([n], ets, [None])
    for sizes in ([[40], [40]], [[3000], [-1]], [[-1], [700]]):
        for sigma in (3, 77, 2**63 + 5):
            say(f"boundary sizes={sizes} sigma={sigma}")
            _, _, ref, got = run_layer_both(olib, [n], ets, [None], [np.array([0])], sizes, sigma,
                                            g=g)
            diffs = compare(ref, got, 1, 1, 2)
            assert not diffs, "\n".join(diffs[:10])


def hubs():
    """Destinations 0 .. 3 with in-degrees 70000 (importance 0 per edge),
    5000, 300 and 0, sources spread over 100000 vertices; two node types so
    that candidates of both types arise."""
    rng = np.random.default_rng(11)
    n0, n1 = 100_000, 3_000
    degs = [70000, 5000, 300, 0]
    idx0 = [np.sort(rng.choice(n0, size=k, replace=False)) for k in degs]
    ip0 = np.concatenate([[0], np.cumsum(degs), np.full(n1 - len(degs), sum(degs))])
    # type-1 destinations from type-0 sources, and type-0 destinations from type 1
    degs1 = [40, 2000] + [0] * (n0 - 2)
    idx1 = [np.sort(rng.choice(n1, size=k, replace=False)) for k in degs1[:2]]
    ip1 = np.concatenate([[0], np.cumsum(degs1)])
    ets = [(0, 1, ip0.astype(np.int64), np.concatenate(idx0).astype(np.int64)),
           (1, 0, ip1.astype(np.int64), np.concatenate(idx1).astype(np.int64))]
    return [n0, n1], ets


@pytest.mark.parametrize("sizes", [[[-1, -1]], [[300, 10], [64, 64]], [[0, 5000], [1, -1]],
                                   [[100000, 0], [2, 2]]])
def test_layer_hubs(olib, sizes):
    nn, ets = hubs()
    g = gpu_graph(nn, ets, [None, None])
    seeds = [np.array([1, 0]), np.array([0, 1, 3, 2])]
    for sigma in (0, 9):
        say(f"hubs sizes={sizes} sigma={sigma}")
        _, _, ref, got = run_layer_both(olib, nn, ets, [None, None], seeds, sizes, sigma, g=g)
        diffs = compare(ref, got, 2, 2, len(sizes))
        assert not diffs, "\n".join(diffs[:10])


def test_layer_errors_and_recovery(olib):
    rng = np.random.default_rng(3)
    nn, ets, feats = W.random_hetero(rng, max_nodes=30, max_deg=10)
    g = gpu_graph(nn, ets, feats)
    T = len(nn)
    seeds = [np.array([0], np.int64) if n > 0 else None for n in nn]
    for bad in ([[-2] * T], [[1] * (T + 1)]):
        with pytest.raises((hg.HGError, ValueError)):
            g.sample_layers(gpu_seeds(seeds), bad, 0)
    t0 = next(t for t in range(T) if nn[t] > 0)
    rep = list(seeds)
    rep[t0] = np.array([0, 0], np.int64)
    with pytest.raises(hg.HGError) as ex:
        g.sample_layers(gpu_seeds(rep), [[1] * T], 0)
    assert ex.value.status == hg.HG_EINVAL
    far = list(seeds)
    far[t0] = np.array([nn[t0]], np.int64)
    with pytest.raises(hg.HGError) as ex:
        g.sample_layers(gpu_seeds(far), [[1] * T], 0)
    assert ex.value.status == hg.HG_EINVAL
    # nine node types (the per-type tables live on the device, not in the launch)
    many_nn = [2] * 9
    many_ets = [(0, 1, np.array([0, 1, 1]), np.array([1])),
                (1, 0, np.array([0, 1, 1]), np.array([0]))]
    many = gpu_graph(many_nn, many_ets, [None] * 9)
    mseeds = [np.array([0])] + [None] * 8
    _, _, mref, mgot = run_layer_both(olib, many_nn, many_ets, [None] * 9, mseeds,
                                      [[1] * 9, [-1] * 9], 3, g=many)
    assert not compare(mref, mgot, 9, 2, 2)
    # the failures left the workspaces clean
    sizes = [[-1] * T, [2] * T]
    _, _, ref, got = run_layer_both(olib, nn, ets, feats, seeds, sizes, 5, g=g)
    diffs = compare(ref, got, T, len(ets), 2)
    assert not diffs, "\n".join(diffs[:10])
    # no hops: the input frontier is the seeds
    b0 = g.sample_layers(gpu_seeds(seeds), [], 0)
    for t in range(T):
        want = np.zeros(0, np.int64) if seeds[t] is None else seeds[t]
        assert np.array_equal(b0.input_nodes(t).cpu().numpy(), want)


@pytest.mark.slow
def test_layer_workload_academic(olib):
    """Layer-wise batches on the academic graph: the workload's 1024 paper
    seeds, 512 draws per node type in each of two hops, every featured type
    gathered."""
    wl = W.WORKLOADS[2]
    gen = W.make_graph(wl, device="cuda")
    g = hg.Graph(list(zip(gen.num_nodes, gen.feats)), gen.etypes)
    host = oracle.HostGraph(gen.host_ntypes(), gen.host_etypes(), lib=olib, check=False)
    sizes = [[k] * g.T for k in W.LAYER_SIZES]
    for bno in range(2):
        seeds = W.seeds_per_type(wl, bno)
        say(f"academic layer batch {bno}")
        b = g.sample_layers(gpu_seeds(seeds), sizes, bno, gather="all")
        got = result_dict(g, b)
        ref = host.sample_layers(seeds, sizes, bno)
        diffs = compare(ref, got, g.T, g.R, len(sizes))
        assert not diffs, "\n".join(diffs[:10])
        for t in range(g.T):
            want = host.gather(t, ref["input"][t])
            assert b.features(t).cpu().numpy().tobytes() == want.tobytes(), f"type {t}"
        say(f"academic layer batch {bno}: equal "
            f"({sum(v[3].size for v in ref['edges'].values())} kept edges)")


@pytest.mark.parametrize("chunk", range(2))
def test_layer_bundles_equal_single_calls(olib, chunk):
    """Every batch of a layer-wise bundle is the batch its own call makes
    (blocks and gathered bytes), and the oracle's."""
    rng = np.random.default_rng(9300 + chunk)
    for c in range(10):
        nn, ets, feats, seeds, sizes, sigma = pins.random_layer_case(rng, max_nodes=60,
                                                                     max_deg=40)
        g = gpu_graph(nn, ets, feats)
        B = [2, 4, 9][c % 3]
        seeds_list = [seeds]
        for b in range(1, B):
            seeds_list.append([None if s is None else
                               rng.choice(nn[t], size=s.size, replace=False).astype(np.int64)
                               for t, s in enumerate(seeds)])
        sigmas = [sigma + 29 * b for b in range(B)]
        say(f"layer bundle chunk {chunk} case {c}: B={B} T={len(nn)} sizes={sizes}")
        bl = g.sample_layers_bundle([gpu_seeds(s) for s in seeds_list], sizes, sigmas,
                                    gather="all")
        assert len(bl) == B
        for b in range(B):
            single = g.sample_layers(gpu_seeds(seeds_list[b]), sizes, sigmas[b], gather="all")
            got = result_dict(g, bl[b])
            diffs = compare(result_dict(g, single), got, len(nn), len(ets), len(sizes))
            assert not diffs, f"case {c} batch {b}: " + "\n".join(diffs[:10])
            for t, f in enumerate(feats):
                if f is not None:
                    assert bl[b].features(t).cpu().numpy().tobytes() == \
                        single.features(t).cpu().numpy().tobytes()
            if b == B - 1:
                ref = oracle.HostGraph(list(zip(nn, feats)), ets, lib=olib).sample_layers(
                    seeds_list[b], sizes, sigmas[b])
                diffs = compare(ref, got, len(nn), len(ets), len(sizes))
                assert not diffs, f"case {c} batch {b} vs oracle: " + "\n".join(diffs[:10])


def sparse_relations(rng, R, n0=300, n1=80):
    """Two node types and R edge types with a handful of edges each: about 3%
    of the destinations of an edge type have 1 to 3 in-edges."""
    nn = [n0, n1]
    ets = []
    for _e in range(R):
        s, d = int(rng.integers(0, 2)), int(rng.integers(0, 2))
        indptr, indices = [0], []
        for _v in range(nn[d]):
            k = int(rng.integers(1, 4)) if rng.random() < 0.03 else 0
            indices.extend(int(x) for x in np.sort(rng.choice(nn[s], size=k, replace=False)))
            indptr.append(len(indices))
        ets.append((s, d, np.array(indptr, np.int64), np.array(indices, np.int64)))
    feats = [rng.standard_normal((n0, 4)).astype(np.float32), None]
    return nn, ets, feats


@pytest.mark.parametrize("R", [6, 40, 70])
def test_layer_many_relations(olib, R):
    """Many sparse edge types: a tile of 2048 in-edges then spans more etypes than
    the kernels' per-tile tables hold (32), and the etype of each edge is searched
    for instead; with 6 a tile spans few.  Single calls and a bundle of 4
    against the oracle."""
    rng = np.random.default_rng(8800 + R)
    nn, ets, feats = many_relations(rng, R) if R <= 6 else sparse_relations(rng, R)
    g = gpu_graph(nn, ets, feats)
    host = oracle.HostGraph(list(zip(nn, feats)), ets, lib=olib)
    for c in range(4):
        seeds = [rng.choice(nn[0], size=int(rng.integers(20, 200)), replace=False).astype(np.int64),
                 rng.choice(nn[1], size=int(rng.integers(0, 30)), replace=False).astype(np.int64)]
        H = int(rng.integers(1, 4))
        sizes = [[[-1, 0, 1, 5, 40][int(rng.integers(0, 5))] for _ in range(2)] for _ in range(H)]
        sigma = int(rng.integers(0, 1 << 63))
        say(f"layer many relations R={R} case {c}: H={H} sizes={sizes}")
        b = g.sample_layers(gpu_seeds(seeds), sizes, sigma, gather="all")
        got = result_dict(g, b)
        ref = host.sample_layers(seeds, sizes, sigma)
        diffs = compare(ref, got, 2, R, H)
        assert not diffs, f"case {c}: " + "\n".join(diffs[:10])
        assert b.features(0).cpu().numpy().tobytes() == feats[0][got["input"][0]].tobytes()
        # four copies of 70 etypes: the next-hop plan scans its 280 etypes in two chunks
        sigmas = [sigma, sigma + 1, sigma + 2, sigma + 3]
        bl = g.sample_layers_bundle([gpu_seeds(seeds)] * 4, sizes, sigmas, gather=[])
        for k in range(4):
            refk = ref if k == 0 else host.sample_layers(seeds, sizes, sigmas[k])
            diffs = compare(refk, result_dict(g, bl[k]), 2, R, H)
            assert not diffs, f"case {c} bundle copy {k}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("total", [1, 63, 64, 65, 2047, 2048, 2049, 4096, 4160, 6145])
@pytest.mark.parametrize("pairs", [1, 3, 700])
def test_layer_edge_tiles(olib, total, pairs):
    """The frontier's in-edges end on, before and after the edges of a flag
    word (64 positions) and of a tile (2048), with few pairs and with many (most
    of one in-edge when there are few).  Kept: none, a few, all."""
    pairs = min(pairs, total)
    rng = np.random.default_rng(100 * total + pairs)
    n = 9000
    deg = np.full(pairs, 1)
    deg[0] += total - pairs - (total - pairs) // 2
    deg[-1] += (total - pairs) // 2
    idx = [np.sort(rng.choice(n, size=k, replace=False)) for k in deg]
    ip = np.concatenate([[0], np.cumsum(deg), np.full(n - pairs, total)]).astype(np.int64)
    ets = [(0, 0, ip, np.concatenate(idx).astype(np.int64))]
    g = gpu_graph([n], ets, [None])
    # the pairs' destinations among others without in-edges
    seeds = [np.concatenate([np.arange(pairs), np.arange(pairs, pairs + 40)])[::-1].copy()]
    for sizes in ([[-1]], [[0]], [[7]], [[300], [5]]):
        _, _, ref, got = run_layer_both(olib, [n], ets, [None], seeds, sizes, total, g=g)
        diffs = compare(ref, got, 1, 1, len(sizes))
        assert not diffs, f"sizes {sizes}: " + "\n".join(diffs[:10])


def bins_graph(n, degs, rng, near):
    """One node type of n vertices; destination k has degs[k] in-edges, half of
    them from vertices next to a multiple of 8192 when `near` (the bins' ends), the
    others from anywhere."""
    ends = np.unique(np.concatenate([np.arange(0, n, 8192) + d for d in (-1, 0, 1)]))
    ends = ends[(ends >= 0) & (ends < n)]
    idx = []
    for k in degs:
        a = rng.choice(ends, size=min(k // 2, ends.size), replace=False) if near else ends[:0]
        rest = rng.choice(n, size=2 * k + 8, replace=False)
        rest = rest[~np.isin(rest, a)][:k - a.size]
        idx.append(np.sort(np.concatenate([a, rest])))
    ip = np.concatenate([[0], np.cumsum(degs), np.full(n - len(degs), sum(degs))])
    return [(0, 0, ip.astype(np.int64), np.concatenate(idx).astype(np.int64))]


@pytest.mark.parametrize("n", [8191, 8192, 8193, 16384, 16385, 40_000])
def test_layer_importance_bins(olib, n):
    """Hops of few in-edges, whose importance is summed by atomics, on the graphs of
    the bins' tests (test_layer_bins_of_large_hops): node types that end on, before
    and after a bitmap tile and half of one, candidates there that are reached by
    several destinations."""
    rng = np.random.default_rng(n)
    degs = [min(3000, n // 3), 500, 40, 3, 1, 1, 0, 700]
    ets = bins_graph(n, degs, rng, True)
    g = gpu_graph([n], ets, [None])
    seeds = [np.array([7, 0, 3, 1, 6, 2, 5, 4, n - 1])]
    for sizes in ([[-1]], [[50]], [[2000], [9]]):
        for sigma in (1, 2**50):
            _, _, ref, got = run_layer_both(olib, [n], ets, [None], seeds, sizes, sigma, g=g)
            diffs = compare(ref, got, 1, 1, len(sizes))
            assert not diffs, f"sizes {sizes}: " + "\n".join(diffs[:10])


def test_layer_more_bins_than_fit(olib):
    """A bundle whose copies make more than 8192 bins sums the importance with
    global atomics whatever its in-edges: each mini-batch equals its own call and two
    equal the oracle."""
    n, B = 2_120_000, 32  # 130 bitmap tiles of two bins each, per copy
    rng = np.random.default_rng(5)
    ets = bins_graph(n, [70_000, 3000, 3000, 40, 1, 5], rng, True)
    g = gpu_graph([n], ets, [None])
    host = oracle.HostGraph([(n, None)], ets, lib=olib)
    sizes = [[300], [-1]]
    seeds = [[rng.permutation(6)[:1 + b % 6].astype(np.int64)] for b in range(B)]
    deg = np.diff(ets[0][2])
    assert sum(int(deg[s[0]].sum()) for s in seeds) >= internal("kBinsFromEdges")
    assert B * -(-n // 16_384) * 2 > internal("kMaxBins")
    bl = g.sample_layers_bundle([gpu_seeds(s) for s in seeds], sizes, list(range(B)), gather=[])
    for b in range(B):
        got = result_dict(g, bl[b])
        one = result_dict(g, g.sample_layers(gpu_seeds(seeds[b]), sizes, b))
        diffs = compare(one, got, 1, 1, 2)
        assert not diffs, f"batch {b}: " + "\n".join(diffs[:10])
        if b in (5, 30):
            diffs = compare(host.sample_layers(seeds[b], sizes, b), got, 1, 1, 2)
            assert not diffs, f"batch {b} vs oracle: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("n,dests", [(8191, 400), (8193, 383), (16384, 400), (40_000, 360)])
def test_layer_bins_of_large_hops(olib, n, dests):
    """The candidates' importance is summed a bin of 8192 vertices at a time from 2^20
    in-edges on (8193 x 383 stays just below in its first hop): node types that end on,
    before and after a bin and a bitmap tile (two bins), sources at the bins' ends."""
    rng = np.random.default_rng(n)
    ets = bins_graph(n, [min(3000, n // 3)] * dests + [40, 1, 0], rng, True)
    g = gpu_graph([n], ets, [None])
    seeds = [np.concatenate([np.arange(dests + 3)[::-1], [n - 1]])]
    for sizes in ([[-1]], [[2000], [9]]):
        _, _, ref, got = run_layer_both(olib, [n], ets, [None], seeds, sizes, 2**50, g=g)
        diffs = compare(ref, got, 1, 1, len(sizes))
        assert not diffs, f"sizes {sizes}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("pairs", [8191, 8192, 8193, 20_000])
@pytest.mark.parametrize("total", [300, 2048, 5000])
def test_layer_tiles_of_empty_pairs(olib, total, pairs):
    """Tiles among many empty pairs: a block finds its positions' pairs by going
    through up to 8192 of them, and of more each position searches.  Pairs that start
    before the tile, on its first position and on its last."""
    rng = np.random.default_rng(total + pairs)
    n = 25_000
    deg = np.zeros(n, np.int64)
    at = np.unique(np.concatenate([[0, 1, pairs // 2], rng.choice(pairs, size=120)]))
    deg[at] = rng.multinomial(total - at.size, np.full(at.size, 1 / at.size)) + 1
    idx = [np.sort(rng.choice(n, size=k, replace=False)) for k in deg if k]
    ets = [(0, 0, np.concatenate([[0], np.cumsum(deg)]).astype(np.int64),
            np.concatenate(idx).astype(np.int64))]
    g = gpu_graph([n], ets, [None])
    seeds = [np.arange(pairs)]
    for sizes in ([[-1]], [[9]], [[200], [-1]]):
        _, _, ref, got = run_layer_both(olib, [n], ets, [None], seeds, sizes, total, g=g)
        diffs = compare(ref, got, 1, 1, len(sizes))
        assert not diffs, f"sizes {sizes}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("records", [32767, 32768, 32769, 65536, 65537, 400_001])
def test_layer_large_bins(olib, records):
    """Bins of more than 32768 records are summed in parts: a type of one full bin
    with as many, one fewer and more; beside it a type of many bins, one of them with
    a candidate from a destination past 65536 in-edges (no importance) and one of
    65536 (importance 1) in every bin.  Twice, as the sums have to be clean again."""
    assert internal("kBinPart") == 32768 and internal("kBinVerts") == 8192
    rng = np.random.default_rng(records)
    nn = [2000, 8192, 50_000]
    deg1 = rng.multinomial(records, np.full(1500, 1 / 1500))
    deg1 = np.concatenate([deg1, np.zeros(nn[0] - 1500, np.int64)])
    deg2 = np.full(nn[0], 450)
    deg2[:4] = [65537, 65536, 70_000, 0]
    ets = [(1, 0, *csc(rng, deg1, nn[1])), (2, 0, *csc(rng, deg2, nn[2]))]
    g = gpu_graph(nn, ets, [None] * 3)
    seeds = [rng.permutation(nn[0]), np.array([5]), None]
    for sizes in ([[-1, -1, -1]], [[0, 40, 3000]], [[0, 40, 3000]]):
        _, _, ref, got = run_layer_both(olib, nn, ets, [None] * 3, seeds, sizes, records, g=g)
        assert frontier_in_edges(ets, ref, 0) >= internal("kBinsFromEdges")
        diffs = compare(ref, got, 3, 2, 1)
        assert not diffs, f"sizes {sizes}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("copies", [1, 3])
def test_layer_bins_of_bundles(olib, copies):
    """Importance by bins over three node types with partial last bins (sizes on and
    off a bin's and a bitmap tile's), and over the copies of a bundle, each keyed as its
    own call: every kind of draw, two hops above the bins' threshold."""
    rng = np.random.default_rng(copies)
    nn = [40_001, 8193, 16_384]
    ets = []
    for s, d, mean in ((0, 0, 40), (1, 0, 30), (2, 0, 35), (0, 1, 50), (2, 1, 3), (1, 2, 20)):
        deg = rng.geometric(1 / mean, size=nn[d]) - 1
        ets.append((s, d, *csc(rng, deg, nn[s])))
    g = gpu_graph(nn, ets, [None] * 3)
    host = oracle.HostGraph([(n, None) for n in nn], ets, lib=olib, check=False)
    n = 16_000 // copies
    for sizes in ([[30, -1, 500], [-1, 7, 0]], [[0, 64, -1], [2000, 2000, 2000]]):
        batches = [[rng.permutation(nn[0])[:n + b], rng.permutation(nn[1])[:n // 4 + 7 * b],
                    rng.permutation(nn[2])[:n // 9]] for b in range(copies)]
        refs = [host.sample_layers(s, sizes, 90 + b) for b, s in enumerate(batches)]
        for h in range(2):
            total = sum(frontier_in_edges(ets, r, h) for r in refs)
            assert total >= internal("kBinsFromEdges")
        bl = g.sample_layers_bundle([gpu_seeds(s) for s in batches], sizes,
                                    [90 + b for b in range(copies)], gather=[])
        for b in range(copies):
            diffs = compare(refs[b], result_dict(g, bl[b]), 3, len(ets), 2)
            assert not diffs, f"sizes {sizes} batch {b}: " + "\n".join(diffs[:10])


def test_layer_bins_past_the_tile_tables(olib):
    """Importance by bins where a tile of positions spans more than 32 edge types and
    more than 8192 pairs (no table of either), between two edge types of full tiles."""
    rng = np.random.default_rng(17)
    nn = [12_000, 30_000]
    full = np.full(nn[0], 60)
    ets = [(1, 0, *csc(rng, full, nn[1]))]
    for _ in range(45):
        deg = np.zeros(nn[0], np.int64)
        deg[rng.choice(nn[0], size=9, replace=False)] = rng.integers(1, 5, size=9)
        ets.append((int(rng.integers(0, 2)), 0, *csc(rng, deg, nn[0])))
    # 45 types of 9000 pairs and some 20 in-edges each: less than a tile together
    assert sum(int(e[2][-1]) for e in ets[1:]) < internal("kEdgeTile")
    ets.append((0, 0, *csc(rng, full, nn[0])))
    g = gpu_graph(nn, ets, [None] * 2)
    seeds = [rng.permutation(nn[0])[:9000], None]
    for sizes in ([[-1, -1]], [[500, 900]]):
        _, _, ref, got = run_layer_both(olib, nn, ets, [None] * 2, seeds, sizes, 4, g=g)
        assert frontier_in_edges(ets, ref, 0) >= internal("kBinsFromEdges")
        diffs = compare(ref, got, 2, len(ets), 1)
        assert not diffs, f"sizes {sizes}: " + "\n".join(diffs[:10])
