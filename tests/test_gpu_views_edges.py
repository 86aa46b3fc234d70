"""Cheap bettors' views at the edges of the kernel's slices (1024 bettors), row
chunks, staged history (120 rows) and settled windows (256): sampled views
against the oracle one by one, counts against the views, and nothing written
outside the rows asked for."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from oracle import bettors as OB
from paper_2108_02419_amd._bbe import Bettors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.mark.parametrize("nb,n,first,n_eval", [(1, 2, 0, 1), (1023, 20, 250, 1), (1024, 7, 0, 9),
                                               (1025, 13, 117, 17), (5000, 20, 119, 200),
                                               (3001, 5, 255, 8), (70_001, 20, 60, 260)])
def test_views_across_slices_rows_and_windows(torch, nb, n, first, n_eval):
    rng = np.random.default_rng([nb, n])
    rows = 400
    tr = np.cumsum(np.float32(rng.uniform(1.0, 9.0, (rows, n))), axis=0, dtype=np.float32)
    L = float(tr.max()) + 50.0
    kinds = rng.integers(0, 4, nb).astype(np.uint8)
    params = np.zeros(nb, np.float32)
    params[kinds == 2] = rng.uniform(0, 60, int((kinds == 2).sum()))
    windows = np.float32([1, 2, 7, 8, 119, 120, 121, 255, 256, 257, 300, 1 << 20])
    params[kinds == 3] = rng.choice(windows, int((kinds == 3).sum()))
    announce(f"views bettors={nb} n={n} rows {first}+{n_eval}")
    pad = 3  # the rows begin at an odd address
    buf = torch.full((pad + n_eval * nb + 64,), 0xEE, dtype=torch.uint8, device="cuda")
    views = buf[pad:pad + n_eval * nb].view(n_eval, nb)
    counts = torch.full((n_eval, n), -1, dtype=torch.int32, device="cuda")
    Bettors(kinds, params).views(torch.from_numpy(tr).cuda(), rows, L, 5, 77, first, n_eval,
                                 views=views, counts=counts)
    torch.cuda.synchronize()
    v, c = views.cpu().numpy(), counts.cpu().numpy()
    assert (buf[:pad] == 0xEE).all() and (buf[pad + n_eval * nb:] == 0xEE).all()
    at = zip(rng.integers(0, n_eval, 600), rng.integers(0, nb, 600))
    for r, b in list(at) + [(0, 0), (n_eval - 1, nb - 1)]:
        want = OB.view(int(kinds[b]), float(params[b]), tr, int(first + r), L, 5, int(b), 77)
        assert v[r, b] == want, (r, b, kinds[b], params[b])
    for r in range(n_eval):
        np.testing.assert_array_equal(np.bincount(v[r], minlength=n), c[r])
