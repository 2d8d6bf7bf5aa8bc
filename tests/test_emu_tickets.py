"""The small kernel's ticket counters, one per event once a batch's launch has 16 groups for
each, on the CPU under the sanitizers: groups of one wave, of several and two per workgroup, with
one and more static rounds before the tickets, an empty event and one in any order among those
that hold a counter; and the first ticket of a single event, drawn from three static rounds on."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2004_04334_amd import synth
from tests.emu import emu
from tests.gpu_util import compare


@pytest.fixture(scope="module")
def emulator(oracle_mod):
    emu.build(sanitizer="address")
    emu.build(sanitizer="thread")
    return oracle_mod


def _event(n_present, n_modules, seed):
    """1-9 digis in each of n_present modules."""
    rng = np.random.default_rng([41, seed])
    mods = np.sort(rng.permutation(n_modules)[:n_present])
    mod = np.repeat(mods, rng.integers(1, 10, n_present))
    lin = np.concatenate([rng.choice(160 * 416, c, replace=False) for c in np.unique(mod, return_counts=True)[1]])
    return synth.from_pixels(mod, lin % 160, lin // 160, n_modules=n_modules, seed=seed)


def _shuffled(ev, seed):
    p = np.random.default_rng(seed).permutation(ev["module"].size)
    return {k: (v[p] if isinstance(v, np.ndarray) else v) for k, v in ev.items()}


# small kernel's workgroups: 64 groups for the four counters of four events
@pytest.mark.parametrize("wg,mpw,grid_s,sanitizer", [(64, 1, 64, "address"), (256, 4, 16, "address"), (128, 1, 64, "address"),
                                                     (256, 2, 64, "address"), (64, 1, 64, "thread"), (128, 1, 64, "thread")])
def test_a_counter_per_event(emulator, wg, mpw, grid_s, sanitizer):
    per_round = grid_s * mpw
    for units in (per_round + 9, 3 * per_round - 1) if sanitizer == "address" else (per_round + 9,):
        n = units // 3                       # three events with modules, of which the lists hold them all
        M = 2 * n + 4
        empty = {k: np.zeros(0, np.uint16) for k in ("module", "row", "col", "adc")}
        evs = [_event(n, M, 1), dict(empty, n_modules=M), _shuffled(_event(n, M, 2), 2), _event(units - 2 * n, M, 3)]
        any_order = [False, False, True, False]
        res = emu.run(evs, M, wg=wg, mpw=mpw, grids=(2, 1, grid_s, 2), header=True, any_order=any_order, sanitizer=sanitizer)
        for i, (r, e) in enumerate(zip(res, evs)):
            compare(r, emulator.cluster_event(e, 2000, any_order=any_order[i]), f"{units} units, event {i}")


@pytest.mark.parametrize("wg,mpw", [(64, 1), (256, 2)])
def test_single_event_draws_from_three_rounds_on(emulator, wg, mpw):
    M = 5 * 3 * mpw                          # five rounds of three workgroups, three of them static
    ev = _event(M - 2, M, 4)
    for fused in (True, False):
        (r,) = emu.run([ev], M, wg=wg, mpw=mpw, grids=(2, 1, 3, 2), fused=fused)
        compare(r, emulator.cluster_event(ev, 2000), f"fused {fused}")
