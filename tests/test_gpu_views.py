"""The tensors over a mini-batch's arrays: their shapes, types and devices, that
each keeps the mini-batch alive, and the accessors' errors."""
import gc

import numpy as np
import pytest
import torch

import paper_2112_15345_amd as hg
from gpu_harness import gpu_graph, gpu_seeds, result_dict

pytestmark = pytest.mark.gpu


def small(dtype):
    nn = [5, 4]
    ets = [(0, 1, np.array([0, 2, 2, 5, 6]), np.array([1, 3, 0, 2, 4, 4])),
           (1, 0, np.zeros(6, np.int64), np.zeros(0, np.int64))]
    feats = [torch.arange(15, dtype=torch.float32).reshape(5, 3).to(dtype).cuda(), None]
    return nn, ets, feats


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
def test_views(dtype):
    nn, ets, feats = small(dtype)
    g = gpu_graph(nn, ets, feats)
    b = g.sample_blocks(gpu_seeds([None, np.array([3, 0, 1])]), [[-1, -1]], 7, gather="all")
    n_dst, gid = b.nodes(0, 0)
    assert n_dst == 0 and gid.dtype == torch.int64 and gid.device == g.etypes[0][2].device
    assert gid.tolist() == [1, 3, 4]
    ip, sl, dl, eid = b.edges(0, 0)
    assert ip.tolist() == [0, 1, 3, 3] and eid.tolist() == [5, 0, 1]
    assert sl.tolist() == [2, 0, 1] and dl.tolist() == [0, 1, 1]
    assert (ip.dtype, sl.dtype, dl.dtype, eid.dtype) == (torch.int64, torch.int32, torch.int32,
                                                         torch.int64)
    # an edge type without kept edges: one closing offset, empty arrays
    ip, sl, dl, eid = b.edges(0, 1)
    assert ip.tolist() == [0] and sl.shape == dl.shape == eid.shape == (0,)
    x = b.features(0)
    assert x.dtype == dtype and x.shape == (3, 3) and torch.equal(x, feats[0][[1, 3, 4]])
    assert b.features(1) is None
    assert b.seeds(1).tolist() == [3, 0, 1] and b.input_nodes(1).tolist() == [3, 0, 1]


def test_views_keep_the_batch():
    nn, ets, feats = small(torch.float32)
    g = gpu_graph(nn, ets, feats)
    b = g.sample_blocks(gpu_seeds([None, np.arange(4)]), [[-1, -1]], 7, gather="all")
    want = result_dict(g, b)
    x, eid = b.features(0), b.edges(0, 0)[3]
    keep = x.clone()
    del b
    gc.collect()
    # batches that would take the freed arrays
    others = [g.sample_blocks(gpu_seeds([None, np.arange(4)[::-1].copy()]), [[2, 1]], s,
                              gather="all") for s in range(20)]
    torch.cuda.synchronize()
    assert torch.equal(x, keep) and eid.cpu().numpy().tolist() == want["edges"][(0, 0)][3].tolist()
    del others, x, eid


@pytest.mark.parametrize("call", [lambda b: b.nodes(1, 0), lambda b: b.nodes(0, 2),
                                  lambda b: b.nodes(0, -1), lambda b: b.edges(0, 2),
                                  lambda b: b.edges(-1, 0), lambda b: b.edges(0, -1),
                                  lambda b: b.input_nodes(2), lambda b: b.features(5),
                                  lambda b: b.seeds(-1), lambda b: b.edge_pairs(0)])
def test_view_errors(call):
    nn, ets, feats = small(torch.float32)
    g = gpu_graph(nn, ets, feats)
    b = g.sample_blocks(gpu_seeds([None, np.arange(4)]), [[-1, -1]], 7, gather="all")
    with pytest.raises(hg.HGError) as ex:
        call(b)
    assert ex.value.status == hg.HG_EINVAL and str(ex.value)
