"""The small kernel's work distribution in batches: one ticket counter per event once a
launch has 16 groups for each, one in all below that, none when a few static rounds cover a
single event.  Batches of 1, 2, 7 and 40 events with empty ones among them, launched again
on the same slots in another order and then one by one, so that a counter left from one
launch would lose or repeat modules of the next; bit-exact against the oracle."""
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


@pytest.mark.parametrize("wg,mpw", [(64, 1), (256, 1), (256, 4), (512, 2)])
@pytest.mark.parametrize("k", [1, 2, 7, 40])
def test_batches_share_out_their_modules(px, k, wg, mpw):
    import torch
    M = 700
    evs = []
    for i in range(k):
        if i % 5 == 3:
            evs.append({n: np.zeros(0, np.uint16) for n in ("module", "row", "col", "adc")})
        else:
            evs.append(synth.async_event(i, n_modules=M) if i % 2 == 0 else
                       synth.batch_event(i, n_modules=M, lo=2000, hi=20000))
    evs = [dict(e, n_modules=M) for e in evs]
    refs = [oracle.cluster_event(e, 2000) for e in evs]
    ctx = px.Context(M, 2000)
    ctx.set_kernel_config(wg, mpw)
    digis = [px.Digis.from_numpy(e, "cuda", any_order=i % 7 == 6) for i, e in enumerate(evs)]
    slots = [px.Event(ctx, 60000) for _ in evs]
    batch = px.Batch(ctx, k)
    stream = torch.cuda.current_stream()
    for turn, (graph, defer) in enumerate(((False, False), (True, False), (False, True), (True, False))):
        order = [(i + turn) % k for i in range(k)]
        px.acquire_batch(batch, slots, [digis[i] for i in order], stream, graph=graph, defer_big=defer)
        px.wait(slots[0])
        for s, i in zip(slots, order):
            compare(px.produce(s).numpy(), refs[i], f"turn {turn} event {i}")
    for i, s in enumerate(slots[:8]):
        px.acquire(s, digis[i], stream)
        px.wait(s)
        compare(px.produce(s).numpy(), refs[i], f"alone {i}")
    batch.close()
    for s in slots:
        s.close()
    ctx.close()
