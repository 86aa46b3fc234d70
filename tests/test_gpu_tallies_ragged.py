"""Finish-order tallies over matrices that start anywhere in memory and end
anywhere in their last 16 bytes: exact against plain counting on the host."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from oracle import orders as O
from paper_2108_02419_amd import api

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.mark.parametrize("n", [1, 2, 5, 6, 7, 13, 16, 20])
def test_any_address_and_length(torch, n):
    rng = np.random.default_rng(n)
    for sims, offset in ((1, 0), (1, 15), (3, 7), (17, 1), (1024, 9), (40_003, 3), (300_000, 16)):
        rows = np.argsort(rng.random((sims, n)), axis=1).astype(np.uint8)
        rows[rng.random(sims) < 0.2, n // 2:] = 0xFF  # places not reached
        announce(f"tallies n={n} sims={sims} offset={offset}")
        buf = torch.zeros(offset + sims * n + 32, dtype=torch.uint8, device="cuda")
        orders = buf[offset:offset + sims * n].view(sims, n)
        orders.copy_(torch.from_numpy(rows))
        rc = api.rank_counts(orders, n)
        pmf = api.order_pmf(orders, n) if n <= 7 else None
        torch.cuda.synchronize()
        np.testing.assert_array_equal(rc.cpu().numpy().astype(np.uint64), O.rank_counts(rows, n))
        if pmf is not None:
            np.testing.assert_array_equal(pmf.cpu().numpy().astype(np.uint64),
                                          O.order_pmf(rows, n))
