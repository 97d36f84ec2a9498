"""How the threads of the in-LDS generation kernel go through their chains,
replayed on the CPU with the kernel's own code (csrc/gen_chains.h): at every
step each chain that has rotations in it is held by its thread, in whole
passes, in the two parts of a split pass and in every segment."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_02840_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("gen_chains") / "driver")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(CSRC, "plan.cpp"), os.path.join(ROOT, "tests", "sanitize", "gen_chains_driver.cpp"),
                    "-o", exe], check=True, timeout=300)
    return exe


# a thread's first and second chain; sizes at which a segment starts with the
# lanes of a wavefront a chain apart and one is due before the rest; the largest
@pytest.mark.parametrize("first,last,stride", [(2, 500, 83), (513, 1600, 181), (2387, 2387, 1), (2405, 2405, 1),
                                               (1700, 3300, 173), (3390, 3392, 1)])
def test_every_chain_is_held_when_it_starts(driver, first, last, stride):
    r = subprocess.run([driver, str(first), str(last), str(stride)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-4000:]
    assert "gen chains: 0 of" in r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("tiling,m,n", [((18, 5, 1), 2387, 2387), ((18, 3, 1), 2414, 2405)])
def test_resumed_segments_match_the_oracle(oracle, tiling, m, n):
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_02840_amd import bdu
    rng = np.random.default_rng(n)
    d, e = rng.uniform(1.0, 10.0, n), rng.uniform(0.0, 1.0, n - 1)
    u, v = rng.standard_normal(m), rng.standard_normal(n)
    I, J = np.asfortranarray(np.eye(m)), np.asfortranarray(np.eye(n))
    old = bdu.get_tiling()
    bdu.set_tiling(*tiling)
    try:
        h = bdu.Handle(I, d, e, J)
    finally:
        bdu.set_tiling(*old)
    h.update_projected(u, v)
    Q, d1, e1, P = h.read()
    h.close()
    rows = [0, 1, n // 2, n - 1]
    Qr, dr, er, Pr = oracle.bgu_pass_rows(m, n, I[rows], d, e, J[rows], u, v)
    for name, x, y in (("d", d1, dr), ("e", e1, er), ("Q", Q[rows], Qr), ("P", P[rows], Pr)):
        assert np.array_equal(x, y), (name, int(np.sum(x != y)))
