"""Generation in device memory with more chains than threads: its ticks, and
(on the GPU) forced passes at sizes that are otherwise generated in LDS."""
import numpy as np
import pytest
import torch  # before the library is loaded, so that both use one HIP runtime

from paper_2509_02840_amd import bdu


@pytest.fixture
def in_device_memory():
    bdu.set_generation_in_lds(False)
    yield
    bdu.set_generation_in_lds(True)


def _entries(side, i):
    if side == 0:
        return [(r, c) for r in (i, i + 1) for c in range(i - 1, i + 4)] + [("u", i), ("u", i + 1)]
    return [(r, c) for c in (i, i + 1) for r in range(i - 2, i + 3)] + [("v", i), ("v", i + 1)]


@pytest.mark.parametrize("m,n", [(130, 129), (300, 300), (560, 550)])
def test_every_chain_starts_at_its_earliest_tick(in_device_memory, m, n):
    """A barrier follows every tick there, so a chain waits for nothing but the rotations before it
    that share an entry with one of its own, and its thread."""
    side, idx, ph, tick = (x.tolist() for x in bdu.plan_rotations(m, n))
    threads = bdu.plan_stats(m, n)["gen_threads"]
    N = n if m == n else n + 1
    chains, prev = [], None
    for s, i, p, t in zip(side, idx, ph, tick):
        if p == 0:
            continue
        pos = 2 * i if s == 0 else 2 * i - 1
        if s == 2 or prev != (p, pos + 3 if p == 1 else pos - 3):
            chains.append((t, []))
        chains[-1][1].append([(N - 1, n), (N, n), ("u", N - 1), ("u", N), ("v", n)] if s == 2 else _entries(s, i))
        prev = (p, pos) if s != 2 else None
    assert len(chains) == bdu.plan_stats(m, n)["chains"]
    last, free = {}, {}
    for c, (start, rotations) in enumerate(chains):
        earliest = free.get(c % threads, 0)
        for q, cells in enumerate(rotations):
            earliest = max([earliest] + [last[x] + 1 - q for x in cells if x in last])
        assert start == earliest, (c, start, earliest)
        for q, cells in enumerate(rotations):
            for x in cells:
                last[x] = start + q
        free[c % threads] = start + len(rotations)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n", [(700, 640), (1500, 1500), (3000, 3000)])
def test_forced_pass_matches_the_oracle(in_device_memory, oracle, m, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n)
    d, e = rng.uniform(1.0, 10.0, n), rng.uniform(0.0, 1.0, n - 1)
    u, v = rng.standard_normal(m), rng.standard_normal(n)
    I, J = np.asfortranarray(np.eye(m)), np.asfortranarray(np.eye(n))
    h = bdu.Handle(I, d, e, J)
    h.update_projected(u, v)
    Q, d1, e1, P = h.read()
    h.close()
    rows = [0, 1, n // 2, n - 1]
    Qr, dr, er, Pr = oracle.bgu_pass_rows(m, n, I[rows], d, e, J[rows], u, v)
    for name, x, y in (("d", d1, dr), ("e", e1, er), ("Q", Q[rows], Qr), ("P", P[rows], Pr)):
        assert np.array_equal(x, y), (name, int(np.sum(x != y)))
