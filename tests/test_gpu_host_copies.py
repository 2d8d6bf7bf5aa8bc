"""Pinned host digis in and results back out: arrays whose bytes end in every remainder of
an 8-byte word, host arrays on and off 8-byte alignment (one kernel moves them, or one copy
command each), new contents in the same host buffers; bit-exact against the oracle."""
from __future__ import annotations

import time

import numpy as np
import pytest

import oracle
from paper_2004_04334_amd import synth
from tests.gpu_util import compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def px():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_04334_amd import pxcl
    pxcl.lib()
    oracle.build()
    return pxcl


@pytest.mark.parametrize("offset", [0, 1, 4])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 1021, 1022, 60001])
def test_pinned_round_trip(px, n, offset):
    import torch
    ctx = px.Context(64, 2000)
    slot = px.Event(ctx, n)
    bufs = [torch.empty(n + offset, dtype=torch.int16, pin_memory=True) for _ in range(4)]
    d = px.Digis(*(b[offset:].view(torch.uint16) for b in bufs))
    dst = px.HostCopy(n, n_digis=n, hits=True)
    for turn in range(3):
        lin = np.random.default_rng([n, turn]).choice(64 * 160 * 416, n, replace=False)
        ev = synth.from_pixels(lin // 66560, lin % 160, lin % 66560 // 160, n_modules=64, seed=turn)
        for b, k in zip(bufs, ("module", "row", "col", "adc")):
            b.numpy()[offset:] = ev[k].view(np.int16)
        ref = oracle.hits(ev, 2000)
        px.acquire(slot, d)
        px.hits_enqueue(slot)
        if turn:
            px.hits_wait(slot)
        f = px.Flag()
        px.copy_to_host(slot, dst, flag=f)
        t0 = time.time()
        while f.fired == 0:
            assert time.time() - t0 < 30
        px.hits_wait(slot)
        got = dst.numpy(n)
        compare(got, ref, f"turn {turn}")
        assert np.array_equal(got["x"], ref["x"]) and np.array_equal(got["y"], ref["y"])
    slot.close()
    ctx.close()
