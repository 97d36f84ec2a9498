"""Tracking updates at the sizes where the products' and residuals' blocks have
edges (64 columns, 8 terms, 32 columns in flight, 64 and 256 rows, one and four
rows a lane), against the oracle: the products
bit for bit, the projections within the bounds of the other tracking tests."""
import pytest

from paper_2509_02840_amd import workloads as W
from tests.test_gpu_track import _lockstep

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bdu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2509_02840_amd import bdu as B
    B.lib()
    return B


@pytest.mark.parametrize("m,n,r", [(9, 7, 2), (65, 64, 7), (257, 255, 31), (256, 300, 33), (520, 130, 64),
                                   (700, 513, 65), (16400, 300, 200)])
def test_tracking_update_at_block_edges(bdu, oracle, m, n, r):
    state = W.tracking_state(m, n, r, 700 + r)
    t = bdu.Tracker(*state)
    for step in range(2):
        b, c = W.tracking_update(m, n, 710 + 7 * step + r)
        state, _ = _lockstep(bdu, oracle, t, state, b, c, f"step {step}")
    t.close()
