"""Host arrays that the copy kernel does not take, and the largest ones it does: non-coherent
pinned memory and pageable memory (a copy command each), 16 MB in total (one kernel) and one
digi more (copy commands); new contents in the same buffers each turn, results copied back into
memory of the same kind, bit-exact against the oracle."""
from __future__ import annotations

import ctypes
import time

import numpy as np
import pytest

import oracle
from paper_2004_04334_amd import synth
from tests.gpu_util import compare

pytestmark = pytest.mark.gpu

NAMES = ("module", "row", "col", "adc")


@pytest.fixture(scope="module")
def px():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_04334_amd import pxcl
    pxcl.lib()
    oracle.build()
    return pxcl


def _event(n, seed, modules=64):
    lin = np.random.default_rng([n, seed]).choice(modules * 160 * 416, n, replace=False)
    return synth.from_pixels(lin // 66560, lin % 160, lin % 66560 // 160, n_modules=modules, seed=seed)


def _round_trip(px, slot, bufs, dst, outs, ev):
    """One event from the arrays `bufs`, its results into `dst`, whose arrays are `outs`."""
    lib, n = px.lib(), ev["module"].size
    for b, k in zip(bufs, NAMES):
        b[:] = ev[k]
    d = px._Digis(*(b.ctypes.data for b in bufs), n, px.WHERE_HOST, 0, 0)
    flags = px.Flag(), px.Flag()
    assert lib.pxcl_acquire(slot.handle, ctypes.byref(d), None, px.flag_cb_ptr(), ctypes.addressof(flags[0])) == px.OK
    px.wait(slot)
    assert lib.pxcl_copy_to_host(slot.handle, None, ctypes.byref(dst), px.flag_cb_ptr(), ctypes.addressof(flags[1])) == px.OK
    t0 = time.time()
    while flags[1].fired == 0:
        assert time.time() - t0 < 30
    k = dst.n_clusters
    got = {"status": dst.status, "n_clusters": k, "id": outs[0][:k], "charge": outs[1][:k], "size": outs[2][:k],
           "digi": outs[3][:n]}
    compare(got, oracle.cluster_event(ev, 2000))


@pytest.mark.parametrize("kind", ["non-coherent", "pageable"])
def test_other_host_memory(px, kind):
    n = 1021
    hip = ctypes.CDLL("libamdhip64.so")
    blocks = []

    def array(dtype):
        if kind == "pageable":
            return np.zeros(n, dtype)
        p = ctypes.c_void_p()
        assert hip.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(4 * n), ctypes.c_uint(0x80000000)) == 0   # hipHostMallocNonCoherent
        blocks.append(p)
        return np.frombuffer((ctypes.c_char * (4 * n)).from_address(p.value), dtype)[:n]

    ctx = px.Context(64, 2000)
    slot = px.Event(ctx, n)
    bufs = [array(np.uint16) for _ in NAMES]
    outs = [array(np.int32) for _ in range(4)]
    dst = px._HostClusters(*(a.ctypes.data for a in outs), None, None, n, 0, px.E_NOT_READY)
    for turn in range(3):
        _round_trip(px, slot, bufs, dst, outs, _event(n, turn))
    slot.close()
    ctx.close()
    for p in blocks:
        hip.hipHostFree(p)


@pytest.mark.parametrize("n", [2 << 20, (2 << 20) + 1])
def test_largest_copies_by_kernel(px, n):
    import torch
    ctx = px.Context(64, 2000)
    slot = px.Event(ctx, n)
    pinned = [torch.empty(n, dtype=torch.int16, pin_memory=True) for _ in NAMES]
    bufs = [t.numpy().view(np.uint16) for t in pinned]
    host = px.HostCopy(n, n_digis=n)
    outs = [t.numpy() for t in (host.id, host.charge, host.size, host.digi)]
    _round_trip(px, slot, bufs, host.s, outs, _event(n, 1))
    slot.close()
    ctx.close()
