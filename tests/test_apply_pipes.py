"""Start chunks of the staged applier with two pipelines (CPU): block b runs on
pipeline b mod 2, and the schedule is replayed as the kernel runs it."""
import os
import subprocess

import numpy as np
import pytest

from tests.test_host_schedule import _pipelined_launch_violations
from paper_2509_02840_amd import bdu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_02840_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include <stdlib.h>
#include "plan.h"
int main(int argc, char **argv)
{
    const int64_t m = atoll(argv[1]), n = atoll(argv[2]);
    auto P = bdu::build_plan(m, n, atoi(argv[3]), atoi(argv[4]), 1024);
    for (int side = 0; side < 2; ++side)
        for (auto &b : P->blocks[side])
            printf("%d %d %d %d %d %d %lld\n", side, b.base, b.lmax, b.nfront, b.phase, b.start2, (long long)b.off);
    return argc != 5;
}
"""


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("pipes")
    (d / "driver.cpp").write_text(DRIVER)
    exe = str(d / "driver")
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC,
                        os.path.join(CSRC, "plan.cpp"), str(d / "driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-2000:]
    return exe


def _memory_order_violations(K0, NW, blocks, ncols):
    """Loads at least DL + 3 fronts after every earlier block's store of the
    column, stores after every earlier block's load and store of it."""
    U = K0 + 3
    DL = U // 3
    stored, loaded, bad = {}, {}, []
    for i, (base, lmax, nfront, phase, start, off) in enumerate(blocks.tolist()):
        if lmax < 0:
            continue
        d = -1 if phase == 1 else 1
        for lam in range(lmax + 2):
            c = base - 1 + d * lam
            if not 0 <= c < ncols:
                continue
            F0 = start * U
            load = F0 + (-1 if lam < 7 else max(-1, (lam - 7) // 3 - DL))
            store = F0 + lam // 3 + (NW - 1) * U + K0
            if load < stored.get(c, -10 ** 9) + DL + 3 or store <= max(stored.get(c, -10 ** 9), loaded.get(c, -10 ** 9)):
                bad.append((i, c))
            stored[c] = store
            loaded[c] = max(loaded.get(c, -10 ** 9), load)
    return bad


@pytest.mark.parametrize("k0,nw", [(12, 7), (12, 15)])
@pytest.mark.parametrize("m,n", [(2, 2), (14, 12), (130, 97), (257, 191), (420, 150), (900, 900)])
def test_two_pipelines_replay(planner, k0, nw, m, n):
    out = subprocess.run([planner, str(m), str(n), str(k0), str(nw)], capture_output=True, text=True)
    assert out.returncode == 0
    rows = np.array([[int(x) for x in line.split()] for line in out.stdout.splitlines()], dtype=np.int64)
    saved = bdu.get_tiling()
    bdu.set_tiling(k0, nw, 1)
    try:
        bcut = bdu.plan_segments(m, n)[1]
    finally:
        bdu.set_tiling(*saved)
    for side, ncols in ((0, m), (1, n)):
        b = rows[rows[:, 0] == side][:, 1:]
        nb1 = int(np.sum(b[:, 3] == 1))
        for lo, hi in ((0, nb1), (nb1, len(b))):  # blocks without work come last in their phase
            live = b[lo:hi, 1] >= 0
            assert np.all(live[:-1] | ~live[1:])
        assert np.all(np.diff(b[:, 4]) >= 0)
        assert _memory_order_violations(k0, nw, b, ncols) == []
        # a run is one phase's blocks of a part; each pipeline of it by itself
        cuts = sorted({0, nb1, len(b)} | {int(c) for c in bcut})
        for lo, hi in zip(cuts, cuts[1:]):
            for p in (0, 1):
                assert _pipelined_launch_violations(k0, nw, b[lo + p:hi:2], ncols) == []


def test_memory_order_checker_sees_one_pipelines_starts(planner):
    """Blocks started as early as their own pipeline allows, whatever the
    other's stores, would load columns too soon."""
    out = subprocess.run([planner, "600", "600", "12", "7"], capture_output=True, text=True).stdout
    rows = np.array([[int(x) for x in line.split()] for line in out.splitlines()], dtype=np.int64)
    b = rows[rows[:, 0] == 0][:, 1:].copy()
    free = [0, 0]
    for i in range(len(b)):
        if b[i, 1] >= 0:
            b[i, 4] = free[i % 2]
            free[i % 2] += ((b[i, 1] + 1) // 3 + 12 - 1 + 15) // 15
    assert _memory_order_violations(12, 7, b, 600) != []
