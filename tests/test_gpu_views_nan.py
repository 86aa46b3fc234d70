"""Cheap bettors' views at trace rows that hold NaN (rows past a trace's end
hold what the caller left there): leader and runner-up as a scan from the first
competitor finds them, each view a competitor of the race, and the counts those
of the views."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from oracle import bettors as OB
from paper_2108_02419_amd._bbe import Bettors

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def _scan(x, skip=-1):
    best = -1
    for c in range(len(x)):
        if c != skip and (best < 0 or x[c] > x[best]):
            best = c
    return best


def _view(kind, param, tr, r, L, t0, b, seed):
    x = tr[r]
    p1 = _scan(x)
    p2 = _scan(x, p1)
    if kind == OB.ZI:
        return OB.zi_pick(seed, t0 + r, b, len(x))
    if kind == OB.UD:
        return p2 if p2 >= 0 and np.float32(x[p1] - x[p2]) < np.float32(param) else p1
    if kind == OB.LINEX:
        moved = x - tr[r - min(int(param), r)] > 0
        return OB.linex_pick(tr, r, int(param), L) if moved.any() else p1
    return p1


@pytest.mark.parametrize("n", [1, 2, 3, 20])
def test_rows_with_nan(torch, n):
    rng = np.random.default_rng(n)
    rows, nb, L = 24, 1500, 400.0
    tr = np.cumsum(np.float32(rng.uniform(1.0, 9.0, (rows, n))), axis=0, dtype=np.float32)
    for r in range(2, rows, 2):  # one, some or all of a row
        tr[r, rng.permutation(n)[:1 + int(rng.integers(0, n))]] = np.nan
    tr[8] = np.nan
    tr[10, 0] = np.nan
    kinds = rng.integers(0, 4, nb).astype(np.uint8)
    params = np.where(kinds == OB.LINEX, rng.integers(1, 30, nb), 4.0).astype(np.float32)
    announce(f"views of rows with NaN, n={n}")
    views = torch.zeros((rows, nb), dtype=torch.uint8, device="cuda")
    counts = torch.zeros((rows, n), dtype=torch.int32, device="cuda")
    Bettors(kinds, params).views(torch.from_numpy(tr).cuda(), rows, L, 3, 11, 0, rows,
                                 views=views, counts=counts)
    torch.cuda.synchronize()
    v, c = views.cpu().numpy(), counts.cpu().numpy()
    with np.errstate(invalid="ignore"):
        for r in range(rows):
            want = [_view(int(kinds[b]), float(params[b]), tr, r, L, 3, b, 11)
                    for b in range(nb)]
            np.testing.assert_array_equal(v[r], want)
            np.testing.assert_array_equal(np.bincount(v[r], minlength=n), c[r])
