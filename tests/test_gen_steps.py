"""Ticks of the in-LDS generation kernel (no device needed).

The kernel orders two rotations of one wavefront by their ticks alone (its
LDS accesses run in order) and two of different wavefronts by a barrier every
STEP ticks, so rotations that share an entry of the working matrix, u or v
must be at later ticks in schedule order, and in a later step when they run
on different wavefronts.  Chain c of a phase (0-based, by its start position)
runs on thread c mod the plan's thread count.
"""
import numpy as np
import pytest

from paper_2509_02840_amd import bdu

STEP, LANES = 8, 64


def _entries(side, i):
    if side == 0:
        return [(r, c) for r in (i, i + 1) for c in range(i - 1, i + 4)] + [("u", i), ("u", i + 1)]
    return [(r, c) for c in (i, i + 1) for r in range(i - 2, i + 3)] + [("v", i), ("v", i + 1)]


def _violations(m, n, tick_of=lambda t, wave: t):
    side, idx, ph, tick = (x.tolist() for x in bdu.plan_rotations(m, n))
    threads = bdu.plan_stats(m, n)["gen_threads"]
    last, bad, prev, chain = {}, [], None, 0
    for s, i, p, t in zip(side, idx, ph, tick):
        if p not in (1, 2):
            prev = None
            continue
        pos = 2 * i if s == 0 else 2 * i - 1
        if prev != (p, pos + 3 if p == 1 else pos - 3):  # a chain starts
            chain = pos - 1 if p == 1 else pos - 2
        prev = (p, pos)
        wave = (chain % threads) // LANES
        t = tick_of(t, wave)
        for cell in _entries(s, i):
            if cell in last:
                t0, p0, w0 = last[cell]
                ok = t > t0 if (p0, w0) == (p, wave) else t // STEP > t0 // STEP
                if not ok:
                    bad.append((p, chain, s, i, t, cell, t0, w0))
            last[cell] = (t, p, wave)
    return bad


# one, two and three chunks of 64 chains, their edges, and sizes whose chains
# outnumber the 1024 threads
@pytest.mark.parametrize("m,n", [(2, 2), (3, 2), (33, 33), (34, 33), (34, 34), (66, 64), (97, 97), (130, 129),
                                 (515, 514), (577, 577), (700, 640)])
def test_steps_order_every_shared_entry(m, n):
    assert _violations(m, n) == []


def test_checker_sees_a_missing_step():
    """Without the delay of one step a chunk, neighbouring wavefronts share entries within a step."""
    assert _violations(200, 200, lambda t, wave: t - STEP * wave) != []
