"""Modules above the small kernel's capacity at the edges of the register and the scratch
mode: sizes around 16,384 digis (the last digis of a group of four missing or not), more
clusters than scratch mode sums in LDS (an even lattice), a checkerboard, a fully fired
module and both serpentines; grouped, in any order and off alignment, with fused hits.
Whole numbers and hits are compared bit-exactly with the oracle."""
from __future__ import annotations

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


def _event():
    rng = np.random.default_rng(31)
    lin = [rng.choice(160 * 416, n, replace=False) for n in (2049, 4097, 16383, 16384, 16385, 16386, 16387, 30001)]
    r, c = np.meshgrid(np.arange(160), np.arange(416), indexing="ij")
    for pick in ((r % 2 == 0) & (c % 2 == 0), (r + c) % 2 == 0, r >= 0, c % 2 == 0, r % 3 != 0):
        lin.append((c * 160 + r)[pick])
    for row_wise in (True, False):
        sr, sc = synth.serpentine(row_wise)
        lin.append(sc * 160 + sr)
    mod = np.concatenate([np.full(x.size, 2 * i) for i, x in enumerate(lin)])
    lin = np.concatenate(lin)
    return synth.from_pixels(mod, lin % 160, lin // 160, n_modules=2 * 15, seed=32)


@pytest.mark.parametrize("any_order,hits,offset", [(False, False, 0), (False, True, 1), (True, True, 3), (True, False, 2)])
def test_large_modules(px, any_order, hits, offset):
    import torch
    ev = _event()
    if any_order:
        p = np.random.default_rng(33).permutation(ev["module"].size)
        ev = {k: (v[p] if isinstance(v, np.ndarray) else v) for k, v in ev.items()}
    ref = oracle.hits(ev, 2000, any_order=any_order)
    d = px.Digis.from_numpy(ev, "cuda", any_order=any_order, hits=hits)
    for k in ("module", "row", "col", "adc"):
        t = torch.empty(d.n + offset, dtype=torch.int16, device="cuda")
        t[offset:] = getattr(d, k).view(torch.int16)
        setattr(d, k, t[offset:].view(torch.uint16))
    ctx = px.Context(30, 2000)
    slot = px.Event(ctx, d.n)
    for _ in range(2):                       # the second time on the slot the first one left
        px.acquire(slot, d, torch.cuda.current_stream())
        px.hits_enqueue(slot, torch.cuda.current_stream())
        px.hits_wait(slot)
        compare(px.produce(slot).numpy(), ref, "large modules")
        h = px.hits_produce(slot).numpy()
        assert np.array_equal(h["x"], ref["x"]) and np.array_equal(h["y"], ref["y"])
    slot.close()
    ctx.close()
