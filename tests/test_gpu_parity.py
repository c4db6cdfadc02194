"""HIP path (through the C ABI) against the CPU oracle, element by element, on
random tiny heterographs and the tiny workload.  All outputs are integers or
copied bits, so the bar is exact equality."""
import ctypes
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2112_15345_amd as hg
import pins
import workloads as W
from gpu_harness import active_rule, many_relations, compare, csc, gpu_graph, gpu_seeds, result_dict

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def olib():
    return oracle.load()


def test_philox_device_matches_oracle(olib):
    rng = np.random.default_rng(1)
    n = 4096
    ctr = rng.integers(0, 1 << 32, size=(n, 4), dtype=np.uint64).astype(np.uint32)
    ctr[0] = 0
    ctr[1] = 0xFFFFFFFF
    key = int(rng.integers(0, 1 << 63)) * 2 + 1
    got = hg.debug_philox(torch.as_tensor(ctr.view(np.int32), device="cuda"), key)
    got = got.cpu().numpy().view(np.uint32)
    for i in range(0, n, 97):
        ref = oracle.philox4x32_10(ctr[i], [key & 0xFFFFFFFF, key >> 32], olib)
        assert np.array_equal(got[i], ref), f"counter {ctr[i]}"
    # and all of them against rocRAND's key definition for the zero-key case
    z = hg.debug_philox(torch.zeros((1, 4), dtype=torch.int32, device="cuda"), 0)
    assert np.array_equal(z.cpu().numpy().view(np.uint32)[0], pins.rr_block(0, 0, 0))


@pytest.mark.parametrize("sigma,hop,etype,lim", [(0, 0, 0, 1 << 31), (2**64 - 1, 2, 5, 123457),
                                                  (987654321, 1, 1199, 0xFFFFFFFF),
                                                  (5, 7, 3, 0)])
def test_key_loop_counts_match_oracle(olib, sigma, hop, etype, lim):
    """The sampler's key loop run alone (hg_bench_philox, the key-rate
    microbenchmark): its count of keys <= lim over edge IDs 0 .. 4n-1 equals
    the oracle's keys of the same edges."""
    n_groups = 64 * 160
    got = int(hg.bench_philox(sigma, hop, etype, n_groups, lim).item())
    keys = np.array([oracle.edge_key(sigma, hop, etype, eid, 32, olib)
                     for eid in range(4 * n_groups)], dtype=np.uint64)
    assert got == int((keys <= lim).sum())
    with pytest.raises(hg.HGError):
        hg.bench_philox(sigma, hop, etype, 100, lim)  # not a multiple of 64


def run_both(olib, nn, ets, feats, seeds, fanouts, sigma, bits):
    g = gpu_graph(nn, ets, feats)
    b = g.sample_blocks(gpu_seeds(seeds), fanouts, sigma, key_bits=bits)
    got = result_dict(g, b)
    ref = oracle.HostGraph(list(zip(nn, feats)), ets, lib=olib).sample_blocks(seeds, fanouts,
                                                                              sigma, bits)
    return g, b, ref, got


@pytest.mark.parametrize("chunk", range(4))
def test_random_heterographs(olib, chunk):
    rng = np.random.default_rng(1000 + chunk)
    for c in range(40):
        case = pins.random_case(rng, max_nodes=60, max_deg=40)
        nn, ets, feats, seeds, fanouts, sigma, bits = case
        say(f"chunk {chunk} case {c}: T={len(nn)} R={len(ets)} H={len(fanouts)} bits={bits}")
        g, b, ref, got = run_both(olib, *case)
        diffs = compare(ref, got, len(nn), len(ets), len(fanouts))
        assert not diffs, f"case {c}: " + "\n".join(diffs[:10])
        fails = pins.check_blocks(nn, ets, seeds, fanouts, sigma, bits, got, brute=False)
        assert not fails, "\n".join(fails[:5])
        # every block's edge count in one call
        assert b.edge_counts() == [[ref["edges"][(h, e)][3].size for e in range(len(ets))]
                                   for h in range(len(fanouts))]
        # gather of the input frontier, every type with features (one call)
        featured = [t for t, f in enumerate(feats) if f is not None]
        allx = g.gather_features_all(b, featured)
        for t in featured:
            assert allx[t].cpu().numpy().tobytes() == feats[t][got["input"][t]].tobytes()
        # and per type
        for t, f in enumerate(feats):
            if f is None:
                with pytest.raises(hg.HGError):
                    g.gather_features(b, t)
                continue
            x = g.gather_features(b, t).cpu().numpy()
            assert x.tobytes() == f[got["input"][t]].tobytes()
        # the fused call: same blocks, and the features it gathered itself
        if bits == 32:
            bf = g.sample_blocks(gpu_seeds(seeds), fanouts, sigma, gather=featured)
            diffs = compare(ref, result_dict(g, bf), len(nn), len(ets), len(fanouts))
            assert not diffs, f"case {c} (fused): " + "\n".join(diffs[:10])
            for t, f in enumerate(feats):
                x = bf.features(t)
                if f is None:
                    assert x is None
                    continue
                assert x.shape == (got["input"][t].size, f.shape[1])
                assert x.cpu().numpy().tobytes() == f[got["input"][t]].tobytes()


def hub_graph(deg, n_src=None, extra=(3, 0, 7)):
    """One node type; destination 0 has `deg` in-edges, a few small ones follow."""
    n_src = n_src or deg + 10
    degs = [deg, *extra]
    indptr = np.concatenate([[0], np.cumsum(degs)]).astype(np.int64)
    rng = np.random.default_rng(deg)
    idx = np.concatenate([np.sort(rng.choice(n_src, size=d, replace=False)) for d in degs])
    n = max(n_src, len(degs))
    indptr = np.concatenate([indptr, np.full(n - len(degs), indptr[-1])]).astype(np.int64)
    return [n], [(0, 0, indptr, idx.astype(np.int64))], [None]


@pytest.mark.parametrize("deg,k,bits", [
    (700, 5, 32), (5000, 25, 32), (70000, 15, 32),      # candidate path
    (3000, 5, 2), (3000, 5, 1), (1200, 600, 32),        # bisection fallback
    (2000, 400, 4), (640, 639, 32), (64, 63, 32), (65, 64, 32),
    # every in-edge kept from more than one chunk's worth: chunked copies
    (70000, -1, 32), (5000, 5000, 32), (2049, 3000, 32), (4097, -1, 32),
])
def test_hub_selection(olib, deg, k, bits):
    nn, ets, feats = hub_graph(deg)
    seeds = [np.array([0, 1, 2, 3], np.int64)]
    for sigma in (0, 1, 2**40 + 3):
        say(f"hub deg={deg} K={k} bits={bits} sigma={sigma}")
        g, b, ref, got = run_both(olib, nn, ets, feats, seeds, [[k], [k]], sigma, bits)
        diffs = compare(ref, got, 1, 1, 2)
        assert not diffs, "\n".join(diffs)


# 16 etypes into a type: the smallest with a mask; 33 and 70: rows of 2 and
# 3 words
@pytest.mark.parametrize("R", [16, 33, 70])
def test_many_relations(olib, R):
    rng = np.random.default_rng(70 + R)
    nn, ets, feats = many_relations(rng, R)
    g = gpu_graph(nn, ets, feats)
    host = oracle.HostGraph(list(zip(nn, feats)), ets, lib=olib)
    for c in range(6):
        seeds = [rng.choice(nn[0], size=int(rng.integers(1, 60)), replace=False).astype(np.int64),
                 rng.choice(nn[1], size=int(rng.integers(0, 10)), replace=False).astype(np.int64)]
        H = int(rng.integers(1, 4))
        fan = [[[-1, 0, 1, 3, 10][int(rng.integers(0, 5))] for _ in range(R)] for _ in range(H)]
        sigma = int(rng.integers(0, 1 << 63))
        say(f"many relations R={R} case {c}: H={H}")
        b = g.sample_blocks(gpu_seeds(seeds), fan, sigma, gather="all")
        got = result_dict(g, b)
        ref = host.sample_blocks(seeds, fan, sigma)
        diffs = compare(ref, got, 2, R, H)
        assert not diffs, f"case {c}: " + "\n".join(diffs[:10])
        assert b.features(0).cpu().numpy().tobytes() == feats[0][got["input"][0]].tobytes()
        # the same batches bundled (the copies share the masks); four copies of
        # 70 etypes: the next-hop plan scans its 280 etypes in two chunks
        bl = g.sample_bundle([gpu_seeds(seeds)] * 4, fan, [sigma + k for k in range(4)],
                             gather=[])
        for k in range(4):
            refk = ref if k == 0 else host.sample_blocks(seeds, fan, sigma + k)
            diffs = compare(refk, result_dict(g, bl[k]), 2, R, H)
            assert not diffs, f"case {c} bundle copy {k}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("bits", [1, 2, 3, 4, 8])
def test_forced_ties(olib, bits):
    rng = np.random.default_rng(77 + bits)
    for c in range(15):
        nn, ets, feats, seeds, fanouts, sigma, _ = pins.random_case(rng, max_nodes=80, max_deg=70)
        say(f"ties bits={bits} case {c}")
        g, b, ref, got = run_both(olib, nn, ets, feats, seeds, fanouts, sigma, bits)
        diffs = compare(ref, got, len(nn), len(ets), len(fanouts))
        assert not diffs, f"case {c}: " + "\n".join(diffs[:10])


def test_tiny_workload_batches(olib):
    wl = W.WORKLOADS[1]
    gen = W.make_graph(wl)
    hgraph = oracle.HostGraph(gen.host_ntypes(), gen.host_etypes(), lib=olib)
    g = hg.Graph([(n, f.cuda()) for n, f in zip(gen.num_nodes, gen.feats)],
                 [(s, d, ip.cuda(), ix.cuda()) for s, d, ip, ix in gen.etypes])
    for bno in range(20):
        seeds = W.seeds_per_type(wl, bno)
        say(f"tiny workload batch {bno}")
        b = g.sample_blocks(gpu_seeds(seeds), wl.fanout_matrix(), bno)
        got = result_dict(g, b)
        ref = hgraph.sample_blocks(seeds, wl.fanout_matrix(), bno)
        diffs = compare(ref, got, g.T, g.R, len(wl.fanouts))
        assert not diffs, f"batch {bno}: " + "\n".join(diffs[:10])
        for t in range(g.T):
            x = g.gather_features(b, t).cpu().numpy()
            assert x.tobytes() == hgraph.gather(t, ref["input"][t]).tobytes()


def test_error_codes_match_oracle(olib):
    indptr = np.array([0, 1, 3, 3], np.int64)
    indices = np.array([2, 0, 1], np.int64)
    g = gpu_graph([3], [(0, 0, indptr, indices)], [None])
    ho = oracle.HostGraph([(3, None)], [(0, 0, indptr, indices)], lib=olib)
    for seeds, fo, kb in [([[1, 1]], [[2]], 32), ([[3]], [[2]], 32), ([[-1]], [[2]], 32),
                          ([[0]], [[-2]], 32), ([[0]], [[1]], 0), ([[0]], [[1]], 33),
                          ([[0, 0]], [], 32)]:
        with pytest.raises(oracle.OracleError) as eo:
            ho.sample_blocks([np.array(seeds[0])], fo, 0, kb)
        with pytest.raises(hg.HGError) as eg:
            g.sample_blocks(gpu_seeds([np.array(seeds[0])]), fo, 0, key_bits=kb)
        assert eo.value.status == eg.value.status == hg.HG_EINVAL
    # a featureless type cannot be gathered, by either call
    b = g.sample_blocks(gpu_seeds([np.array([0])]), [[1]], 0)
    with pytest.raises(hg.HGError):
        g.gather_features(b, 0)
    for gl in ([0], [1], [-1]):
        with pytest.raises(hg.HGError) as e:
            g.sample_blocks(gpu_seeds([np.array([0])]), [[1]], 0, gather=gl)
        assert e.value.status == hg.HG_EINVAL
    with pytest.raises(ValueError):
        g.sample_blocks(gpu_seeds([np.array([0])]), [[1]], 0, key_bits=8, gather=[])
    # invalid CSC arrays are refused at creation
    for ip, ix in [(np.array([0, 1, 3, 2]), indices), (indptr, np.array([2, 0, 3])),
                   (np.array([1, 1, 3, 3]), indices)]:
        with pytest.raises(hg.HGError) as e:
            gpu_graph([3], [(0, 0, ip, ix)], [None])
        assert e.value.status == hg.HG_EINVAL
    # the graph still works after failed calls (map and bitmap left clean)
    b = g.sample_blocks(gpu_seeds([np.array([1, 0])]), [[-1], [-1]], 3)
    got = result_dict(g, b)
    ref = ho.sample_blocks([np.array([1, 0])], [[-1], [-1]], 3)
    assert not compare(ref, got, 1, 1, 2)


def test_zero_hops_and_empty_seeds(olib):
    rng = np.random.default_rng(5)
    nn, ets, feats = W.random_hetero(rng, max_types=2, max_nodes=30)[:3]
    seeds = [np.arange(min(3, n), dtype=np.int64) for n in nn]
    for fanouts in ([], [[2] * len(ets)]):
        g, b, ref, got = run_both(olib, nn, ets, feats, seeds, fanouts, 9, 32)
        assert not compare(ref, got, len(nn), len(ets), len(fanouts))
    empty = [np.zeros(0, np.int64) for _ in nn]
    g, b, ref, got = run_both(olib, nn, ets, feats, empty, [[3] * len(ets)] * 2, 1, 32)
    assert not compare(ref, got, len(nn), len(ets), 2)


def test_determinism_and_two_streams(olib):
    wl = W.WORKLOADS[1]
    gen = W.make_graph(wl)
    g = hg.Graph([(n, f.cuda()) for n, f in zip(gen.num_nodes, gen.feats)],
                 [(s, d, ip.cuda(), ix.cuda()) for s, d, ip, ix in gen.etypes])
    seeds = gpu_seeds(W.seeds_per_type(wl, 3))
    first = result_dict(g, g.sample_blocks(seeds, wl.fanout_matrix(), 3))
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(s1):
        b1 = g.sample_blocks(seeds, wl.fanout_matrix(), 3, stream=s1)
    with torch.cuda.stream(s2):
        b2 = g.sample_blocks(seeds, wl.fanout_matrix(), 3, stream=s2)
    torch.cuda.synchronize()
    for b in (b1, b2):
        assert not compare(first, result_dict(g, b), g.T, g.R, 2)


def test_allocator_failure_releases_everything(olib):
    """An allocator that fails after a few allocations: HG_ENOMEM, every block
    it handed out is returned, and the graph keeps working."""
    state = {"live": {}, "budget": 0, "allocs": 0}

    def alloc(ctx, nbytes, stream):
        if state["allocs"] >= state["budget"]:
            return None
        state["allocs"] += 1
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        state["live"][t.data_ptr()] = t
        return t.data_ptr()

    def free(ctx, ptr, stream):
        state["live"].pop(ptr)

    a = hg.Allocator(None, hg.ALLOC_FN(alloc), hg.FREE_FN(free))
    rng = np.random.default_rng(3)
    nn, ets, feats = W.random_hetero(rng, max_types=2, max_nodes=40)[:3]
    nts = [(n, None if f is None else torch.as_tensor(f).cuda()) for n, f in zip(nn, feats)]
    g = hg.Graph(nts, [(s, d, torch.as_tensor(ip).cuda(), torch.as_tensor(ix).cuda())
                       for s, d, ip, ix in ets], allocator=a)
    seeds = [np.arange(min(4, n), dtype=np.int64) for n in nn]
    fo = [[3] * len(ets)] * 3
    ref = oracle.HostGraph(list(zip(nn, feats)), ets, lib=olib).sample_blocks(seeds, fo, 11)
    for budget in range(0, 12):
        state.update(budget=budget, allocs=0)
        try:
            b = g.sample_blocks(gpu_seeds(seeds), fo, 11)
        except hg.HGError as e:
            assert e.status == hg.HG_ENOMEM
            torch.cuda.synchronize()
            assert not state["live"], f"budget {budget}: {len(state['live'])} blocks leaked"
            continue
        got = result_dict(g, b)
        assert not compare(ref, got, len(nn), len(ets), 3)
        del b
        torch.cuda.synchronize()
        assert not state["live"]
        break
    else:
        pytest.fail("sampling never succeeded")


def expected_keys(ets, ref, fanouts):
    """Keys the sampler must evaluate per hop: the in-degree of every
    (frontier vertex, edge type) pair that keeps K of more than K in-edges."""
    out = []
    for h, row in enumerate(fanouts):
        k = 0
        for e, (s, d, ip, ix) in enumerate(ets):
            nd, sg = ref["nodes"][(h, d)]
            deg = ip[sg[:nd] + 1] - ip[sg[:nd]]
            if row[e] >= 0:
                k += int(deg[deg > row[e]].sum())
        out.append(k)
    return out


def test_block_counts_and_keys(olib):
    """hg_blocks_counts: per-hop frontier and source sizes equal the oracle's,
    and the sampler's key count equals the in-degrees of the pairs that
    select (a bundle reports the sum over its batches)."""
    rng = np.random.default_rng(31)
    for c in range(6):
        nn, ets, feats, seeds, fanouts, sigma, bits = pins.random_case(rng, max_nodes=300,
                                                                       max_deg=3000)
        g, b, ref, got = run_both(olib, nn, ets, feats, seeds, fanouts, sigma, 32)
        nd, ns, keys = b.counts()
        for h in range(len(fanouts)):
            for t in range(len(nn)):
                assert nd[h, t] == ref["nodes"][(h, t)][0]
                assert ns[h, t] == ref["nodes"][(h, t)][1].size
        assert list(keys) == expected_keys(ets, ref, fanouts), f"case {c}"
    wl = W.WORKLOADS[1]
    gen = W.make_graph(wl)
    host = oracle.HostGraph(gen.host_ntypes(), gen.host_etypes(), lib=olib)
    g = hg.Graph([(n, f.cuda()) for n, f in zip(gen.num_nodes, gen.feats)],
                 [(s, d, ip.cuda(), ix.cuda()) for s, d, ip, ix in gen.etypes])
    fan = wl.fanout_matrix()
    batches = [3, 4, 5]
    got = g.sample_bundle([gpu_seeds(W.seeds_per_type(wl, x)) for x in batches], fan, batches)
    want = np.zeros(len(fan), np.int64)
    for x in batches:
        ref = host.sample_blocks(W.seeds_per_type(wl, x), fan, x)
        want += expected_keys(gen.host_etypes(), ref, fan)
    for blocks in got:
        assert list(blocks.counts()[2]) == list(want)


@pytest.mark.parametrize("pad", [0, 3_000_000])
def test_reached_bit_mode(olib, pad):
    """Hops whose kept edges are few next to the graph's vertices mark reached
    sources with bits (atomicOr) instead of bytes; the tiny workload with and
    without 3M isolated extra vertices of each type (every hop in bit mode,
    or a mix) equals the oracle, blocks and gathered bytes."""
    wl = W.WORKLOADS[1]
    gen = W.make_graph(wl)
    nn = [n + pad for n in gen.num_nodes]
    ets = []
    for s, d, ip, ix in gen.host_etypes():
        ets.append((s, d, np.concatenate([ip, np.full(pad, ip[-1], np.int64)]), ix))
    feats = [np.concatenate([f, np.zeros((pad,) + f.shape[1:], f.dtype)])
             for _, f in gen.host_ntypes()]
    g = gpu_graph(nn, ets, feats)
    host = oracle.HostGraph(list(zip(nn, feats)), ets, lib=olib)
    fan = wl.fanout_matrix()
    for b in range(3):
        seeds = W.seeds_per_type(wl, b)
        blocks = g.sample_blocks(gpu_seeds(seeds), fan, b, gather="all")
        ref = host.sample_blocks(seeds, fan, b)
        diffs = compare(ref, result_dict(g, blocks), g.T, g.R, len(fan))
        assert not diffs, f"pad {pad} batch {b}: " + "\n".join(diffs[:5])
        for t in range(g.T):
            assert blocks.features(t).cpu().numpy().tobytes() == \
                host.gather(t, ref["input"][t]).tobytes()
    # a bundle of 4 on the same graph (the virtual graph has 4x the vertices)
    got = g.sample_bundle([gpu_seeds(W.seeds_per_type(wl, b)) for b in range(4)], fan,
                          list(range(4)))
    for b, blocks in enumerate(got):
        ref = host.sample_blocks(W.seeds_per_type(wl, b), fan, b)
        assert not compare(ref, result_dict(g, blocks), g.T, g.R, len(fan))


@pytest.mark.parametrize("R", [16, 31, 32, 33, 64, 65, 130])
def test_mask_bits_of_the_frontier(olib, R):
    """Node types with a non-empty mask, on hops of so few pairs that they go through
    every pair all the same (the larger ones, over the listed pairs, are in
    test_gpu_active_pairs.py): most pairs are empty.  Frontiers that end on, before
    and after a wavefront's 64 vertices, edge types on, before and after a mask
    word's 32; two such node types; single calls and a bundle."""
    rng = np.random.default_rng(300 + R)
    nn = [400, 150]
    ets = []
    for e in range(2 * R):
        d = e & 1
        s = int(rng.integers(0, 2))
        indptr, indices = [0], []
        for _v in range(nn[d]):
            k = int(rng.integers(1, 7)) if rng.random() < 0.1 else 0
            indices.extend(int(x) for x in np.sort(rng.choice(nn[s], size=k, replace=False)))
            indptr.append(len(indices))
        ets.append((s, d, np.array(indptr, np.int64), np.array(indices, np.int64)))
    g = gpu_graph(nn, ets, [None, None])
    host = oracle.HostGraph([(n, None) for n in nn], ets, lib=olib)
    fan = [[3] * (2 * R), [2] * (2 * R)]
    batches = []
    for n0, n1 in ((1, 0), (63, 1), (64, 64), (65, 63), (128, 149), (129, 0)):
        batches.append([rng.choice(nn[0], size=n0, replace=False).astype(np.int64),
                        rng.choice(nn[1], size=n1, replace=False).astype(np.int64)])
    refs = [host.sample_blocks(s, fan, 5 + b) for b, s in enumerate(batches)]
    for b, s in enumerate(batches):
        got = result_dict(g, g.sample_blocks(gpu_seeds(s), fan, 5 + b))
        diffs = compare(refs[b], got, 2, 2 * R, 2)
        assert not diffs, f"seeds {[x.size for x in s]}: " + "\n".join(diffs[:10])
    bl = g.sample_bundle([gpu_seeds(s) for s in batches], fan,
                         [5 + b for b in range(len(batches))], gather=[])
    for b in range(len(batches)):
        diffs = compare(refs[b], result_dict(g, bl[b]), 2, 2 * R, 2)
        assert not diffs, f"bundle batch {b}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("n0", [4095, 4096, 4161])
def test_mask_bits_of_large_hops(olib, n0):
    """A call whose first hop goes through every pair (2^18 of them, one frontier
    vertex fewer and some more) and whose second, the frontier having grown, works on
    the active ones."""
    R, n = 64, 12_000
    rng = np.random.default_rng(n0)
    ets = []
    for _e in range(R):
        deg = np.where(rng.random(n) < 0.05, rng.integers(1, 7, n), 0)
        idx = [np.sort(rng.choice(n, size=k, replace=False)) for k in deg if k]
        ets.append((0, 0, np.concatenate([[0], np.cumsum(deg)]).astype(np.int64),
                    np.concatenate(idx).astype(np.int64)))
    seeds = [rng.permutation(n)[:n0].astype(np.int64)]
    _, _, ref, got = run_both(olib, [n], ets, [None], seeds, [[3] * R, [2] * R], 9, 32)
    active = active_rule([n], ets)
    assert not active([[n0]]) and active([[int(ref["nodes"][(1, 0)][0])]])
    diffs = compare(ref, got, 1, R, 2)
    assert not diffs, "\n".join(diffs[:10])


# key bits for which a hub's candidate list (about K + 4 sqrt(K) + 16 entries, at
# most 512) holds equal keys: several to a value, pairs of them, hardly any; lists
# of 1 to 3 entries past a multiple of four, and of several per lane
@pytest.mark.parametrize("deg,K,bits", [(3000, 20, 12), (3000, 20, 16), (2049, 1, 12),
                                        (2049, 2, 14), (5000, 3, 20), (70000, 300, 14),
                                        (70000, 380, 20), (70000, 100, 32)])
def test_hub_equal_keys(olib, deg, K, bits):
    nn, ets, feats = hub_graph(deg)
    for sigma in range(6):
        _, _, ref, got = run_both(olib, nn, ets, feats, [np.array([0, 3, 1], np.int64)], [[K]],
                                  sigma, bits)
        diffs = compare(ref, got, 1, 1, 1)
        assert not diffs, f"sigma {sigma}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("n", [1, 510, 511, 512, 513, 1023, 1024, 1025, 1500])
def test_small_call_limits(olib, n):
    """Seeds on and around the limits of a one-block start (1024) and of a
    counting pass that publishes its own sizes (one tile: 511 pairs and the end),
    over two hops and again after calls that failed, which leave the frontier bits
    to be cleared."""
    rng = np.random.default_rng(n)
    nn = [1600, 900]
    ets = []
    for s, d in ((0, 0), (1, 0), (0, 1)):
        deg = rng.integers(0, 9, size=nn[d])
        idx = [np.sort(rng.choice(nn[s], size=k, replace=False)) for k in deg]
        ets.append((s, d, np.concatenate([[0], np.cumsum(deg)]).astype(np.int64),
                    np.concatenate(idx).astype(np.int64)))
    g = gpu_graph(nn, ets, [None, None])
    host = oracle.HostGraph([(k, None) for k in nn], ets, lib=olib)
    fan = [[3, 2, 4], [2, 0, -1]]
    for split in (n, n // 2):
        seeds = [rng.choice(nn[0], size=split, replace=False).astype(np.int64),
                 rng.choice(nn[1], size=min(n - split, 900), replace=False).astype(np.int64)]
        ref = host.sample_blocks(seeds, fan, n)
        for again in range(2):
            diffs = compare(ref, result_dict(g, g.sample_blocks(gpu_seeds(seeds), fan, n)), 2, 3, 2)
            assert not diffs, f"split {split} call {again}: " + "\n".join(diffs[:10])
            for bad in (nn[0], -1, seeds[0][0] if split > 1 else nn[0]):
                wrong = [seeds[0].copy(), seeds[1]]
                if split:
                    wrong[0][-1] = bad
                    with pytest.raises(hg.HGError) as ex:
                        g.sample_blocks(gpu_seeds(wrong), fan, n)
                    assert ex.value.status == hg.HG_EINVAL


@pytest.mark.parametrize("n", [40_000, 4_300_000])
def test_new_vertices_by_shares(olib, n):
    """The compaction numbers a wavefront's new vertices a lane per share of 64
    vertices, or a share at a time when some share has more new vertices than there
    are shares with any, or than 17: shares and vertices on either side of both
    limits, full shares, and the last vertices of the type; in the compaction of one
    launch and of three."""
    rng = np.random.default_rng(3)
    cases = []
    for shares in (1, 2, 16, 17, 18, 63, 64):
        for per in (1, 2, 15, 16, 17, 18, 19, 64):
            cases.append((shares, per))
    idx = []
    for shares, per in cases:
        at = np.sort(rng.choice(64, size=shares, replace=False)) + 64 * int(rng.integers(0, 9))
        v = np.concatenate([64 * s + np.sort(rng.choice(64, size=per, replace=False)) for s in at])
        idx.append(np.unique(np.concatenate([v, rng.integers(0, n, size=3), [n - 1]])))
    deg = [x.size for x in idx]
    ip = np.concatenate([[0], np.cumsum(deg), np.full(n - len(deg), sum(deg))]).astype(np.int64)
    ets = [(0, 0, ip, np.concatenate(idx).astype(np.int64))]
    g = gpu_graph([n], ets, [None])
    host = oracle.HostGraph([(n, None)], ets, lib=olib)
    for k in range(0, len(cases), 1 if n < 100_000 else 9):
        seeds = [np.array([k, n - 5], np.int64)]
        diffs = compare(host.sample_blocks(seeds, [[-1]], 1),
                        result_dict(g, g.sample_blocks(gpu_seeds(seeds), [[-1]], 1)), 1, 1, 1)
        assert not diffs, f"{cases[k]}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("sizes", [(2_097_151, 0, 1), (2_097_152, 3, 0), (1, 2_200_000, 1023),
                                   (1024, 1024, 2_100_000, 1, 1, 5000)])
def test_relabel_of_many_edges(olib, sizes):
    """From 2097152 edges on, a block of the relabel takes 1024 of them: edge types
    that end within a block, on its edge and one before, with empty ones between."""
    rng = np.random.default_rng(len(sizes))
    n = 30_000
    ets = []
    for total in sizes:
        deg = np.full(200, total // 200)
        deg[:total % 200] += 1
        ip = np.concatenate([[0], np.cumsum(deg), np.full(n - 200, total)]).astype(np.int64)
        ets.append((0, 0, ip, rng.integers(0, n, size=total).astype(np.int64)))
    g = gpu_graph([n], ets, [None])
    seeds = [rng.permutation(250).astype(np.int64)]
    fan = [[-1] * len(sizes)]
    ref = oracle.HostGraph([(n, None)], ets, lib=olib, check=False).sample_blocks(seeds, fan, 2)
    diffs = compare(ref, result_dict(g, g.sample_blocks(gpu_seeds(seeds), fan, 2)), 1, len(sizes),
                    1)
    assert not diffs, "\n".join(diffs[:10])


@pytest.mark.parametrize("n", [65535, 65536, 65537, 66047, 66048, 66560])
def test_large_counting_pass(olib, n):
    """Hops of 262144 pair slots and more are counted in tiles of 2048 read in
    stripes: edge types that start on, before and after a tile's first pair, an empty
    one at the end (its start is the end of the pairs), the last tile nearly empty and
    full; pairs of every role among them."""
    rng = np.random.default_rng(n)
    nn = [70_000, 10]
    ets = []
    for d in (0, 0, 0, 0, 1):
        deg = rng.choice([0, 1, 2, 7, 14], size=nn[d], p=[0.3, 0.4, 0.2, 0.08, 0.02])
        if d == 0:
            deg[rng.choice(nn[0], size=30, replace=False)] = 40
            deg[rng.choice(nn[0], size=3, replace=False)] = 3000
        ip = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
        ets.append((0, d, ip, rng.integers(0, nn[0], size=ip[-1]).astype(np.int64)))
    g = gpu_graph(nn, ets, [None, None])
    seeds = [rng.permutation(nn[0])[:n].astype(np.int64), None]
    for fan in ([[3, -1, 10, 2, 5]], [[20, 0, 5, 1, 1]]):
        ref = oracle.HostGraph([(k, None) for k in nn], ets, lib=olib,
                               check=False).sample_blocks(seeds, fan, n)
        diffs = compare(ref, result_dict(g, g.sample_blocks(gpu_seeds(seeds), fan, n)), 2, 5, 1)
        assert not diffs, f"{fan}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("copies", [18, 19, 25, 26])
def test_large_counting_pass_of_many_edge_types(olib, copies):
    """A bundle's copies make 1296, 1368, 1800 (the most whose table is held in LDS,
    81 KB with the stripes) and 1872 edge types, none with a mask, at 262144 pair slots
    and more; edge types of few pairs, some of none."""
    rng = np.random.default_rng(copies)
    T = 8
    nn = [9000, 800, 3000, 2500, 700, 3000, 2500, 40]
    ets = [(int(rng.integers(0, T)), d) for d in range(T) for _ in range(9)]
    ets = [(s, d, *csc(rng, rng.choice([0, 1, 3, 20, 60], size=nn[d], p=[.4, .3, .2, .08, .02]),
                       nn[s])) for s, d in ets]
    g = gpu_graph(nn, ets, [None] * T)
    host = oracle.HostGraph([(n, None) for n in nn], ets, lib=olib, check=False)
    per = 262_144 // (9 * copies) + 40
    batches = []
    for b in range(copies):
        n = [per - 230 - 7 * b, 0, 90 + b, 60, 40 + 2 * b, 3, 37, b % 3]
        n[0] += per + 60 - sum(n)
        batches.append([rng.permutation(nn[t])[:n[t]] for t in range(T)])
    assert sum(9 * s.size for x in batches for s in x) >= 262_144
    fan = [[int(rng.choice([-1, 0, 2, 10])) for _ in ets]]
    bl = g.sample_bundle([gpu_seeds(s) for s in batches], fan, list(range(copies)), gather=[])
    for b in (0, 1, copies // 2, copies - 1):
        diffs = compare(host.sample_blocks(batches[b], fan, b), result_dict(g, bl[b]), T, len(ets), 1)
        assert not diffs, f"batch {b}: " + "\n".join(diffs[:10])
