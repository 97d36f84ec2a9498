"""Staged applier: a launch of more than 128 blocks of a phase runs them in
several runs, each with a block table of its own (one pipeline and two).
Sampled rows of Q and P, d and e equal the oracle's bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bdu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_02840_amd import bdu as B
    B.lib()
    return B


# K = 36: 2 (n - 1) / 36 blocks in phase 1; K = 84, two pipelines
@pytest.mark.parametrize("tiling,m,n", [((12, 3, 1), 2330, 2330), ((12, 3, 1), 4700, 2350), ((12, 7, 1), 5420, 5420)])
def test_unsegmented_pass_of_many_blocks(bdu, oracle, tiling, m, n):
    rng = np.random.default_rng(m)
    d, e = rng.uniform(1.0, 10.0, n), rng.uniform(0.0, 1.0, n - 1)
    u, v = rng.standard_normal(m), rng.standard_normal(n)
    I, J = np.asfortranarray(np.eye(m)), np.asfortranarray(np.eye(n))
    old = bdu.get_tiling()
    bdu.set_tiling(*tiling)
    bdu.set_split_pass(0)
    try:
        assert sum(1 for b in bdu.plan_blocks(m, n, 0) if b[3] == 1) > 128
        h = bdu.Handle(I, d, e, J)
    finally:
        bdu.set_split_pass(True)
        bdu.set_tiling(*old)
    h.update_projected(u, v)
    Q, d1, e1, P = h.read()
    h.close()
    rows = [0, 1, n // 2, n - 1]
    Qr, dr, er, Pr = oracle.bgu_pass_rows(m, n, I[rows], d, e, J[rows], u, v)
    for name, x, y in (("d", d1, dr), ("e", e1, er), ("Q", Q[rows], Qr), ("P", P[rows], Pr)):
        assert np.array_equal(x, y), (name, int(np.sum(x != y)))
