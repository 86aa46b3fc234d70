"""Batched in-play states from races with and without a time term, from the
start and from a state, next to each other: every form of a request's record,
in both entry points, equal bit for bit to the oracle."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from paper_2108_02419_amd import _bbe, inputs

pytestmark = pytest.mark.gpu
L = inputs.TRACK_LEN


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


@pytest.mark.parametrize("fn", ["prefix_batch", "prefix_batch_noalloc"])
@pytest.mark.parametrize("B", [1, 4, 37, 97])
def test_records_of_every_form(torch, orc, fn, B):
    rng = np.random.default_rng(B)
    reqs = []
    for i in range(B):
        n = 1 + (7 * i) % 20
        comp = inputs.competitor_params(rng, n)
        if i % 2 == 0:
            comp = inputs.pace_params(rng, comp)
        state = None
        if i % 4 < 2:
            state = orc.race_prefix(comp, L, 1, i, 0, 400.0)
        reqs.append((comp, state, 1200.0 + i))
    specs = [(_bbe.Race(c, L), st, 0, 1, 50 + i, 0) for i, (c, st, _) in enumerate(reqs)]
    out = (torch.zeros(B, dtype=torch.int32, device="cuda"),
           torch.full((B, 20), -7.0, device="cuda"), torch.full((B, 20), -7.0, device="cuda"))
    announce(f"{fn} of {B} requests")
    getattr(_bbe, fn)(specs, np.arange(B), [t for _, _, t in reqs], 3, *out)
    T, P, S = (x.cpu().numpy() for x in out)
    for i, (comp, st, target) in enumerate(reqs):
        n = comp.shape[0]
        t, p, s = orc.race_prefix(comp, L, 3, 50 + i, i, np.float32(target), state=st)
        assert T[i] == t
        np.testing.assert_array_equal(P[i, :n], p)
        np.testing.assert_array_equal(S[i, :n], s)
        assert not P[i, n:].any() and not S[i, n:].any()
