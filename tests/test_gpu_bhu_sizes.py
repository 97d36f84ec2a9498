"""The Householder update at the sizes where its products change shape: chunks
of 128 columns, rows around 64 and 256, and past 512 columns (two passes)."""
import numpy as np
import pytest

from paper_2509_02840_amd import workloads as W

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


@pytest.fixture(scope="module")
def bdu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_02840_amd import bdu as B
    B.lib()
    return B


# the tolerance of the repository's other comparison of this update: n steps
# of sums over n terms
@pytest.mark.parametrize("m,n", [(4, 2), (63, 63), (128, 127), (131, 129), (258, 130), (256, 256), (600, 260),
                                 (520, 515)])
def test_householder_update_at_the_edges(bdu, oracle, m, n):
    f = W.factorization(m, n, 900 + m)
    rng = np.random.default_rng(901 + n)
    b, c = rng.standard_normal(m), rng.standard_normal(n)
    h = bdu.Handle(f.Q, f.d, f.e, f.P)
    h.update_householder(b, c)
    Q, d, e, P = h.read()
    h.close()
    Qo, do, eo, Po = oracle.bhu_update(f.Q, f.d, f.e, f.P, b, c)
    tol = 32 * U * n * n
    scale = np.linalg.norm(f.dense() + np.outer(b, c))
    assert np.abs(d - do).max() <= tol * scale
    assert np.abs(e - eo).max() <= tol * scale
    assert np.abs(Q - Qo).max() <= tol
    assert np.abs(P - Po).max() <= tol
