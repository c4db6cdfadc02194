"""The native module that makes a mini-batch's tensors, when making one fails: the
error is raised and nothing of the mini-batch is kept.  CPU only: the accessors are
stand-ins that give an address that belongs to no device."""
import ctypes
import sys

import pytest

import paper_2112_15345_amd as hg

I64P = ctypes.POINTER(ctypes.c_int64)
PP = ctypes.POINTER(ctypes.c_void_p)
NOWHERE = 0x1000
BIG = 1 << 40  # a count that Python keeps as an object of its own


@ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, I64P, I64P, PP)
def nodes(h, hop, t, n_dst, n_src, gid):
    if n_dst:
        n_dst[0] = BIG
    if n_src:
        n_src[0] = 8
    if gid:
        gid[0] = NOWHERE
    return 0


@ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_int32, I64P, PP)
def one_array(h, t, n, p):
    n[0] = 8
    p[0] = NOWHERE
    return 0


@pytest.fixture()
def views():
    hg.load_library()
    real = hg._accessors(hg._lib)
    fake = list(real)
    fake[0] = ctypes.cast(nodes, ctypes.c_void_p).value
    fake[2] = fake[3] = fake[4] = ctypes.cast(one_array, ctypes.c_void_p).value
    hg._views.bind(*fake)
    yield hg._views
    hg._views.bind(*real)


@pytest.mark.parametrize("call", [lambda v, o: v.nodes(1, 0, 0, -1, o),
                                  lambda v, o: v.input_nodes(1, 0, -1, o),
                                  lambda v, o: v.seeds(1, 0, -1, o),
                                  lambda v, o: v.features(1, 0, 4, hg.HG_DT_F32, -1, o)])
def test_a_failed_tensor_keeps_nothing(views, call):
    class Owner:
        pass

    owner = Owner()
    with pytest.raises(RuntimeError):  # (what a first failure sets up stays)
        call(views, owner)
    refs, blocks = sys.getrefcount(owner), sys.getallocatedblocks()
    for _ in range(300):
        try:
            call(views, owner)
        except RuntimeError:
            pass
    assert sys.getrefcount(owner) == refs
    assert sys.getallocatedblocks() - blocks < 100
