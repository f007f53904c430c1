"""Device buffers shorter than a search needs are refused: the call returns
GRAND_E_DEVICE and no kernel reads or writes past them.  (Every access of a
call that did use one stays within the allocation's 4 KB page.)"""
import ctypes

import numpy as np
import pytest

from parity import say
from workloads import IndexConfig

pytestmark = pytest.mark.gpu

NQ, K, DIM = 4, 10, 64
SIZES = dict(queries=NQ * DIM, ids=NQ * K * 4, dists=NQ * K * 4)


@pytest.mark.parametrize("via", ["index", "reader"])
@pytest.mark.parametrize("short", [None, *SIZES])
def test_short_device_buffers_are_refused(short, via):
    import torch

    from paper_2608_21163_amd import GrandIndex
    from paper_2608_21163_amd.grand import E_DEVICE, E_STATE, OK, Reader

    say(f"[short buffers] {via}, short: {short}")
    torch.cuda.init()
    x = np.random.default_rng(3).integers(0, 256, (200, DIM), np.uint8)
    g = GrandIndex.from_config(IndexConfig("vamana", "u8", "l2", DIM, 200, 16, 32), max_batch=200)
    g.insert(np.arange(200, dtype=np.uint32), x)
    want = g.search(x[:NQ], K, 32)
    r = Reader(g)
    lib, ptr = g.lib, {}
    for name, size in SIZES.items():
        ptr[name] = ctypes.c_void_p()
        # one query's row or one result less than the call needs
        less = 0 if name != short else DIM if name == "queries" else 4
        assert lib.hipMalloc(ctypes.byref(ptr[name]), ctypes.c_size_t(size - less)) == 0
    if short != "queries":
        q = np.ascontiguousarray(x[:NQ])
        assert lib.hipMemcpy(ptr["queries"], ctypes.c_void_p(q.ctypes.data), ctypes.c_size_t(q.nbytes), 4) == 0
    call, h = (lib.grand_search, g.h) if via == "index" else (lib.grand_reader_search, r.h)
    rc = call(h, ptr["queries"], NQ, K, 32, ptr["ids"], ptr["dists"])
    assert rc == (E_DEVICE if short else OK)
    if short is None:
        ids = np.zeros((NQ, K), np.uint32)
        assert lib.hipMemcpy(ctypes.c_void_p(ids.ctypes.data), ptr["ids"], ctypes.c_size_t(ids.nbytes), 4) == 0
        assert np.array_equal(ids, want[0])
    elif via == "index":  # a HIP failure poisons the handle
        assert call(h, ptr["queries"], NQ, K, 32, ptr["ids"], ptr["dists"]) == E_STATE
    r.close()
    g.close()
    for p in ptr.values():
        assert lib.hipFree(p) == 0
