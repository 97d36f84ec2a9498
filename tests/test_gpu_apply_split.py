"""The staged applier's splits on the GPU: every rows-per-panel and pipeline
count its launch rule can pick, at sizes around the panels' edges, against the
oracle bit for bit."""
import numpy as np
import pytest

from paper_2509_02840_amd import workloads as W

pytestmark = pytest.mark.gpu


def _eq(what, x, y):
    np.testing.assert_array_equal(np.asarray(x), np.asarray(y), err_msg=what)


@pytest.fixture(scope="module")
def bdu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_02840_amd import bdu as B
    B.lib()
    return B


# panels of 64 rows (m and n in panels each) decide the split: at most 8, at
# most 62, at most 83 (K = 180), more
@pytest.mark.parametrize("tk", [(12, 7, 1), (12, 15, 1)])
@pytest.mark.parametrize("m,n,split", [(17, 16, 0), (193, 191, 1), (256, 256, 0), (257, 256, 1), (321, 315, 0),
                                       (1991, 211, 0), (3969, 65, 1), (4033, 40, 0), (5200, 70, 0)])
def test_splits_bit_exact(bdu, oracle, tk, m, n, split):
    rng = np.random.default_rng(181 + m + n)
    d, e = rng.uniform(1.0, 10.0, n), rng.uniform(0.0, 1.0, n - 1)
    u, v = rng.standard_normal(m), rng.standard_normal(n)
    I, J = np.asfortranarray(np.eye(m)), np.asfortranarray(np.eye(n))
    saved = bdu.get_tiling()
    bdu.set_tiling(*tk)
    bdu.set_split_pass(split)
    try:
        h = bdu.Handle(I, d, e, J)
        h.update_projected(u, v)
        got = h.read()
        h.close()
    finally:
        bdu.set_tiling(*saved)
        bdu.set_split_pass(True)
    # every row where m is small, else the first, the last and some between
    qr = np.arange(m) if m <= 400 else np.unique(np.r_[0:22, rng.choice(m, 40, replace=False), m - 22:m])
    Qr, dr, er, Pr = oracle.bgu_pass_rows(m, n, I[qr], d, e, J, u, v)
    for nm, x, y in zip("QdeP", (got[0][qr], *got[1:]), (Qr, dr, er, Pr)):
        _eq(f"{tk} {nm}", x, y)


@pytest.mark.parametrize("tk", [(12, 7, 1), (12, 15, 1)])
@pytest.mark.parametrize("count", [2, 9, 33])
def test_batch_splits_match_single(bdu, tk, count):
    """The same handles in a batch, where more panels pick another split."""
    saved = bdu.get_tiling()
    bdu.set_tiling(*tk)
    try:
        fs = [W.factorization(200 + 13 * (i % 5), 150 + 7 * (i % 3), i) for i in range(count)]
        one = [bdu.Handle(f.Q, f.d, f.e, f.P) for f in fs]
        many = [bdu.Handle(f.Q, f.d, f.e, f.P) for f in fs]
    finally:
        bdu.set_tiling(*saved)
    rng = np.random.default_rng(count)
    Bs = [np.asfortranarray(rng.standard_normal((f.Q.shape[0], 1 + i % 2))) / 15 for i, f in enumerate(fs)]
    Cs = [np.asfortranarray(rng.standard_normal((f.P.shape[0], 1 + i % 2))) / 12 for i, f in enumerate(fs)]
    bdu.update_batched(many, Bs, Cs)
    for a, b, B, C in zip(one, many, Bs, Cs):
        a.update(B, C)
        for nm, x, y in zip("QdeP", a.read(), b.read()):
            _eq(nm, x, y)
        a.close()
        b.close()
