"""Generation in LDS at the sizes where its kernel can go wrong: the row
capacities of its instances, chunks of 64 chains, chains outnumbering the
1024 threads, the largest size that fits in LDS, segmented and unsplit
passes, and operands that leave the range of the shortened rotation (zeros,
tiny and huge entries) at chain starts, inside chains and at their ends.  d,
e and sampled rows of Q and P equal the oracle's bit for bit."""
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


def _check(bdu, oracle, m, n, d, e, u, v, rows=4, factors=True):
    """One projected pass from Q = P = I."""
    I, J = np.asfortranarray(np.eye(m)), np.asfortranarray(np.eye(n))
    h = bdu.Handle(I, d, e, J)
    h.update_projected(u, v)
    Q1, d1, e1, P1 = h.read()
    h.close()
    rng = np.random.default_rng(m + n)
    qr, pr = (np.sort(rng.choice(k, min(rows, k), replace=False)) for k in (m, n))
    Qr, dr, er, Pr = oracle.bgu_pass_rows(m, n, I[qr], d, e, J[pr], u, v)
    for name, x, y in (("d", d1, dr), ("e", e1, er), ("Q", Q1[qr], Qr), ("P", P1[pr], Pr))[: 4 if factors else 2]:
        assert np.array_equal(x, y, equal_nan=True), (name, int(np.sum(x != y)))


def _draw(m, n, seed):
    rng = np.random.default_rng(seed)
    return rng, rng.uniform(1.0, 10.0, n), rng.uniform(0.0, 1.0, n - 1), rng.standard_normal(m), rng.standard_normal(n)


@pytest.mark.parametrize("m,n", [(33, 33), (34, 33), (34, 34), (65, 64), (97, 96), (128, 128), (128, 127), (129, 128),
                                 (256, 256), (257, 256), (512, 512), (513, 512), (514, 514), (640, 577), (1024, 1024),
                                 (1025, 1024), (2064, 2064), (2065, 2064), (2450, 2450), (3392, 3392), (3393, 3392)])
@pytest.mark.parametrize("split", [2, 0])
def test_capacities_and_chunks(bdu, oracle, m, n, split):
    if split == 0 and n > 1024:
        pytest.skip("the unsplit pass is covered at the smaller sizes")
    _, d, e, u, v = _draw(m, n, m)
    bdu.set_split_pass(split)
    try:
        _check(bdu, oracle, m, n, d, e, u, v)
    finally:
        bdu.set_split_pass(True)


@pytest.mark.parametrize("kind", ["zeros", "tiny", "huge", "mixed", "nonfinite"])
@pytest.mark.parametrize("m,n", [(40, 40), (150, 101), (560, 560)])
def test_operands_out_of_range(bdu, oracle, m, n, kind):
    rng, d, e, u, v = _draw(m, n, 7 * m + n)
    if kind == "zeros":  # a replaced row on a sparse factorization
        u[:] = 0.0
        u[m // 3] = 1.0
        v[rng.random(n) < 0.8] = 0.0
        e[rng.random(n - 1) < 0.5] = 0.0
    elif kind == "tiny":
        d, e, u, v = d * 2.0 ** -520, e * 2.0 ** -520, u * 2.0 ** -260, v * 2.0 ** -260
    elif kind == "huge":
        d, e, u, v = d * 2.0 ** 500, e * 2.0 ** 500, u * 2.0 ** 250, v * 2.0 ** 250
    elif kind == "mixed":
        d *= 2.0 ** rng.integers(-420, 420, n)
        v *= 2.0 ** rng.integers(-420, 420, n)
        u[rng.random(m) < 0.3] = 0.0
    else:
        v[n // 2] = np.inf
    with np.errstate(all="ignore"):
        # the appliers' identity slots spread a NaN to columns the oracle does
        # not touch: only the generated d and e are compared then
        _check(bdu, oracle, m, n, d, e, u, v, factors=kind != "nonfinite")
