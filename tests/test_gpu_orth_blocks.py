"""Gram matrix and correction step on the GPU at the sizes where their blocks
and steps have edges (columns around multiples of 4, 16, 32, 64 and 128),
against the oracle's plain products.

Tolerances (u = 2^-53, gamma_m = m u / (1 - m u)): an entry of E = X^T X - I
differs by at most 2 gamma_m between two orders of summation, the drifts by at
most 2 gamma_m k, and the corrected factor by at most gamma_m sqrt(m) (rows of
norm about 1) plus the last subtraction's rounding on each side."""
import numpy as np
import pytest

from paper_2509_02840_amd import workloads as W

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def gamma(m):
    return m * U / (1 - m * U)


@pytest.fixture(scope="module")
def bdu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_02840_amd import bdu as B
    B.lib()
    return B


@pytest.mark.parametrize("m,n", [(2, 2), (5, 3), (17, 15), (33, 32), (63, 61), (65, 64), (129, 66), (190, 127),
                                 (257, 129), (385, 384)])
def test_drift_and_correction_at_block_edges(bdu, oracle, m, n):
    f = W.factorization(m, n, 7 * m + n)
    rng = np.random.default_rng(m + n)
    Q = np.asfortranarray(f.Q + 1e-8 * rng.standard_normal((m, m)) / np.sqrt(m))
    P = np.asfortranarray(f.P + 1e-8 * rng.standard_normal((n, n)) / np.sqrt(n))
    h = bdu.Handle(Q, f.d, f.e, P)
    drift = h.reorthogonalize(0.0)
    Q1, _, _, P1 = h.read()
    h.close()
    for g, X, Y, k in ((drift[0], Q, Q1, m), (drift[1], P, P1, n)):
        want = oracle.orth_error(X)
        assert abs(g - want) <= 2 * gamma(k) * k + 1e-12 * want
        assert np.all(np.abs(Y - oracle.reorth_step(X)) <= gamma(k) * np.sqrt(k) + 4 * U * np.abs(X))
