"""Contexts of more modules than the detector of the workloads: above 4,096 the grouping of digis
in any order has no module histogram in LDS and a table kernel of its own, and from 5,120 on a
single event at the 256-thread shape has three static rounds and hands out the rest of its modules
by ticket.  Sparse events with modules above the small kernel's capacity in both modes of the
big-module kernel; grouped and shuffled, alone, in batches and deferred, with hits; launched again
on the same slots.  Bit-exact against the oracle."""
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


def _event(M, seed, fill=0.85):
    """1-9 digis in most modules (the last one among them), 3,000 and 17,000 in two."""
    rng = np.random.default_rng([43, M, seed])
    count = np.where(rng.random(M) < fill, rng.integers(1, 10, M), 0)
    count[M - 1] = 5
    count[M // 3], count[M // 2] = 3000, 17000
    mod = np.repeat(np.arange(M), count)
    lin = np.concatenate([rng.choice(160 * 416, c, replace=False) if c > 100 else rng.choice(400, c, replace=False) * 7
                          for c in count[count > 0]])
    return synth.from_pixels(mod, lin % 160, lin // 160, n_modules=M, seed=seed)


def _shuffled(ev, seed):
    p = np.random.default_rng(seed).permutation(ev["module"].size)
    return {k: (v[p] if isinstance(v, np.ndarray) else v) for k, v in ev.items()}


def _hits(px, slot, ref, what):
    px.hits_enqueue(slot)
    px.hits_wait(slot)
    h = px.hits_produce(slot).numpy()
    assert np.array_equal(h["x"], ref["x"]) and np.array_equal(h["y"], ref["y"]), what


@pytest.mark.parametrize("wg,mpw", [(256, 1), (64, 1)])
@pytest.mark.parametrize("M", [4096, 4097, 5000, 8000, 32263])
def test_single_events(px, M, wg, mpw):
    ev = _event(M, 1)
    mixed = _shuffled(ev, 2)
    refs = oracle.hits(ev, 2000), oracle.hits(mixed, 2000, any_order=True)
    ctx = px.Context(M, 2000)
    ctx.set_kernel_config(wg, mpw)
    slot = px.Event(ctx, ev["module"].size)
    for turn in range(2):
        for any_order, e, ref in ((False, ev, refs[0]), (True, mixed, refs[1])):
            for hits, defer in ((False, False), (True, False), (False, True)):
                what = f"turn {turn} any order {any_order} hits {hits} defer {defer}"
                px.acquire(slot, px.Digis.from_numpy(e, "cuda", any_order=any_order, hits=hits, defer_big=defer))
                px.wait(slot)
                compare(px.produce(slot).numpy(), ref, what)
                _hits(px, slot, ref, what)
    slot.close()
    ctx.close()


@pytest.mark.parametrize("graph", [False, True])
def test_batches(px, graph):
    import torch
    M = 5000
    evs = [_event(M, 3), _shuffled(_event(M, 4), 4), {k: np.zeros(0, np.uint16) for k in ("module", "row", "col", "adc")},
           _shuffled(_event(M, 5, fill=0.1), 5), _event(M, 6, fill=0.1)]
    evs = [dict(e, n_modules=M) for e in evs]
    any_order = [False, True, True, True, False]
    refs = [oracle.cluster_event(e, 2000, any_order=a) for e, a in zip(evs, any_order)]
    ctx = px.Context(M, 2000)
    slots = [px.Event(ctx, max(e["module"].size for e in evs)) for _ in evs]
    digis = [px.Digis.from_numpy(e, "cuda", any_order=a) for e, a in zip(evs, any_order)]
    batch = px.Batch(ctx, len(evs))
    for turn in range(3):
        order = [(i + turn) % len(evs) for i in range(len(evs))]
        px.acquire_batch(batch, slots, [digis[i] for i in order], torch.cuda.current_stream(), graph=graph)
        px.wait(slots[0])
        for s, i in zip(slots, order):
            compare(px.produce(s).numpy(), refs[i], f"turn {turn} event {i}")
    batch.close()
    for s in slots:
        s.close()
    ctx.close()
