"""Hops that work on the active (vertex, edge type) pairs, those whose bit in a
non-empty mask is set, against the CPU oracle: every kind of mini-batch, single and
bundled, at sizes that the rule sends there (checked) and on its other side."""
import numpy as np
import pytest
import torch

import oracle
import pins
from gpu_harness import (active_rule, compare, compare_edges, csc, edge_result_dict, frontier_in_edges,
                         gpu_graph, gpu_seeds, internal, result_dict)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def olib():
    return oracle.load()


def sparse_type(rng, n_dst, n_src, share, most=6):
    """An edge type with in-edges (1 .. most) at a share of its destinations."""
    deg = np.where(rng.random(n_dst) < share, rng.integers(1, most + 1, n_dst), 0)
    return csc(rng, deg, n_src)


def masked_graph(rng, R, nn, share, most=6):
    """R edge types into each of node types 0 and 1 (both with a mask) and three into
    type 2 (without one)."""
    into = [0, 1] * R + [2]
    into[1:1] = into[R:R] = [2]
    ets = []
    for d in into:
        s = int(rng.integers(0, 3))
        ets.append((s, d, *sparse_type(rng, nn[d], nn[s], 0.8 if d == 2 else share, most)))
    return ets


def sizes(seeds):
    return [0 if s is None else s.size for s in seeds]


@pytest.mark.parametrize("R", [17, 31, 32, 33, 64, 65, 130])
def test_frontier_edges(olib, R):
    """The frontier's mask rows are transposed 64 vertices and 64 edge types at a
    time: frontiers that end on, before and after a wavefront's 64 vertices, edge
    types on, before and after a mask word's 32; two types with a mask and one
    without; single calls and bundles, whose copies' pairs start anywhere in a word."""
    rng = np.random.default_rng(300 + R)
    per = 700_000 // R // 64  # 64-vertex groups of the two types' frontiers together
    nn = [64 * per * 2 // 3 + 500, 64 * per // 3 + 500, 900]
    ets = masked_graph(rng, R, nn, 0.05)
    n_et = len(ets)
    g = gpu_graph(nn, ets, [None] * 3)
    host = oracle.HostGraph([(n, None) for n in nn], ets, lib=olib, check=False)
    fan = [[3] * n_et, [2] * n_et]
    shift = ((-1, 1, 63), (0, 0, 64), (1, -1, 65))
    batches = []
    for d0, d1, n2 in shift:
        n = (64 * (per * 2 // 3) + d0, 64 * (per // 3) + d1, n2)
        batches.append([rng.permutation(nn[t])[:n[t]] for t in range(3)])
    for b, s in enumerate(batches):
        assert active_rule(nn, ets)([sizes(s)])
        ref = host.sample_blocks(s, fan, 5 + b)
        diffs = compare(ref, result_dict(g, g.sample_blocks(gpu_seeds(s), fan, 5 + b)), 3, n_et, 2)
        assert not diffs, f"seeds {sizes(s)}: " + "\n".join(diffs[:10])
    parts = [[x[:x.size // 3 + k] for x in s] for k, s in enumerate(batches)]
    assert active_rule(nn, ets)([sizes(s) for s in parts])
    bl = g.sample_bundle([gpu_seeds(s) for s in parts], fan, [5, 6, 7], gather=[])
    for b, s in enumerate(parts):
        diffs = compare(host.sample_blocks(s, fan, 5 + b), result_dict(g, bl[b]), 3, n_et, 2)
        assert not diffs, f"bundle batch {b}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("share", [0.01, 0.2, 0.5])
def test_rule_edges(olib, share):
    """The last frontier that goes through every pair and the first that lists the
    active ones; with half of them active none does."""
    R, n = 64, 24_000
    rng = np.random.default_rng(int(100 * share))
    ets = [(0, 0, *sparse_type(rng, n, n, share, 4)) for _ in range(R)]
    g = gpu_graph([n], ets, [None])
    host = oracle.HostGraph([(n, None)], ets, lib=olib, check=False)
    active = active_rule([n], ets)
    first = next((m for m in range(1, n + 1) if active([[m]])), None)
    if share == 0.5:
        assert first is None
        first = n
    order = rng.permutation(n)
    for m in (first - 1, first):
        s = [order[:m]]
        diffs = compare(host.sample_blocks(s, [[2] * R], m),
                        result_dict(g, g.sample_blocks(gpu_seeds(s), [[2] * R], m)), 1, R, 1)
        assert not diffs, f"{m} seeds: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("copies", [1, 2])
@pytest.mark.parametrize("most", [5, 150])
def test_layers(olib, most, copies):
    """Layer-wise hops over active pairs: importance by atomics (few in-edges) and by
    bins (2^20 and more), the block CSC from the pairs' bits, kept edges' destinations
    through the list; types with a mask and without one."""
    R = 40
    rng = np.random.default_rng(most + copies)
    nn = [16_000, 5000, 700]
    ets = masked_graph(rng, R, nn, 0.05, most)
    n_et = len(ets)
    g = gpu_graph(nn, ets, [None] * 3)
    host = oracle.HostGraph([(n, None) for n in nn], ets, lib=olib, check=False)
    k = copies
    batches = [[rng.permutation(nn[0])[:12_000 // k + b], rng.permutation(nn[1])[:4000 // k - b],
                rng.permutation(nn[2])[:65]] for b in range(k)]
    assert active_rule(nn, ets)([sizes(s) for s in batches])
    for draws in ([[-1, 70, 0], [9, 9, 9]], [[500, -1, -1]], [[0, 0, 3]]):
        H = len(draws)
        refs = [host.sample_layers(s, draws, 31 + b) for b, s in enumerate(batches)]
        total = sum(frontier_in_edges(ets, r, 0) for r in refs)
        assert (total >= internal("kBinsFromEdges")) == (most == 150)
        bl = g.sample_layers_bundle([gpu_seeds(s) for s in batches], draws,
                                    [31 + b for b in range(k)], gather=[])
        for b in range(k):
            diffs = compare(refs[b], result_dict(g, bl[b]), 3, n_et, H)
            assert not diffs, f"draws {draws} batch {b}: " + "\n".join(diffs[:10])


@pytest.mark.parametrize("copies", [1, 2])
def test_edge_seeds_with_exclusion(olib, copies):
    """Link-prediction batches whose hops list their active pairs: excluded edges are
    looked up by pair, a target's and its reverse's, also in pairs that keep all of
    their remaining in-edges and in those that none is left of."""
    rng = np.random.default_rng(copies)
    n, base = 30_000, 20
    # (no parallel edges: a target's reverse is the one edge back)
    fwd = []
    for _ in range(base):
        deg = np.where(rng.random(n) < 0.04, rng.integers(1, 7, n), 0)
        idx = [np.sort(rng.choice(n, size=k, replace=False)) for k in deg if k]
        fwd.append((0, 0, np.concatenate([[0], np.cumsum(deg)]).astype(np.int64),
                    np.concatenate(idx).astype(np.int64)))
    ets, rev_et, rev_eid = pins.with_reverses([n], fwd)
    R = len(ets)
    g = gpu_graph([n], ets, [None])
    host = oracle.HostGraph([(n, None)], ets, lib=olib, check=False)
    batches = []
    for b in range(copies):
        tg = [None] * R
        for e in (0, 3, R - 1):
            tg[e] = rng.permutation(ets[e][3].size)[:4000 - 500 * copies + b].astype(np.int64)
        batches.append(tg)
    dev = lambda xs: [None if x is None else torch.as_tensor(x, device="cuda") for x in xs]
    fan = [[2] * R, [3] * R]
    refs = [host.sample_edge_blocks(tg, fan, 8 + b, n_neg=1, exclude=2, rev_etype=rev_et,
                                    rev_eid=rev_eid) for b, tg in enumerate(batches)]
    assert active_rule([n], ets)([[r["seeds"][0].size] for r in refs])
    bl = g.sample_edge_bundle([dev(tg) for tg in batches], fan, [8 + b for b in range(copies)],
                              n_neg=1, exclude=2, rev_etype=rev_et, rev_eid=dev(rev_eid))
    for b in range(copies):
        diffs = compare_edges(refs[b], edge_result_dict(g, bl[b]), 1, R, 2)
        assert not diffs, f"batch {b}: " + "\n".join(diffs[:10])


def test_many_node_types(olib):
    """More node types with edges into them, over the copies of a bundle, than a row of
    the grid that makes their pairs' bits: one of them with a mask and most of the pairs."""
    rng = np.random.default_rng(12)
    T, R, copies = 60, 40, 20
    nn = [4000] + [30] * (T - 1)
    ets = [(int(rng.integers(0, T)), 0) for _ in range(R)]
    ets += [(int(rng.integers(0, T)), t) for t in range(1, T)]
    ets = [(s, d, *sparse_type(rng, nn[d], nn[s], 0.05 if d == 0 else 0.5)) for s, d in ets]
    n_et = len(ets)
    g = gpu_graph(nn, ets, [None] * T)
    host = oracle.HostGraph([(n, None) for n in nn], ets, lib=olib, check=False)
    batches = [[rng.permutation(nn[0])[:900 + b]] + [rng.permutation(30)[:t % 4]
               for t in range(1, T)] for b in range(copies)]
    assert copies * T > 1024 and active_rule(nn, ets)([sizes(s) for s in batches])
    fan = [[2] * n_et]
    bl = g.sample_bundle([gpu_seeds(s) for s in batches], fan, list(range(copies)), gather=[])
    for b in (0, 1, 11, 17, 19):
        diffs = compare(host.sample_blocks(batches[b], fan, b), result_dict(g, bl[b]), T, n_et, 1)
        assert not diffs, f"batch {b}: " + "\n".join(diffs[:10])
