"""The bench's measured traffic is reported only for the sources it was taken
on: its digest covers every source that the staged applier is compiled from
and the host code that plans and issues its launches (CPU)."""
import os
import re

import bench

CSRC = "paper_2509_02840_amd/csrc"


def _with_includes(name, seen):
    if name not in seen:
        seen.add(name)
        with open(os.path.join(bench.ROOT, CSRC, name)) as f:
            for inc in re.findall(r'^#include "([^"]+)"', f.read(), flags=re.M):
                _with_includes(inc, seen)
    return seen


def test_digest_covers_the_applier():
    files = os.listdir(os.path.join(bench.ROOT, CSRC))
    units = [f for f in files if f.endswith(".hip") and "apply_kernel.h" in _with_includes(f, set())]
    assert len(units) >= 3
    needed = set()
    for f in units:
        needed |= _with_includes(f, set())
    needed |= {"plan.cpp", "bdu.cpp"}
    assert needed <= {os.path.basename(f) for f in bench.TRAFFIC_SOURCES}
