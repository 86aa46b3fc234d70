"""GPU parity of the single-simulation kernels (a lane per competitor): in-play
states of mixed batches and traces, where teams of different sizes share a
wave, draws are made some ticks ahead, positions tie, and races end at once.
Bit for bit against the oracle."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from paper_2108_02419_amd import _bbe, api, inputs

pytestmark = pytest.mark.gpu
L = inputs.TRACK_LEN


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def _request(rng, n, i):
    """(comp, state, target) of one request, of one of six kinds."""
    comp = inputs.competitor_params(rng, n)
    comp[:, 4] = rng.choice([0.0, 2.0, 40.0], size=n)
    state, target = None, float(rng.uniform(1.0, 1950.0))
    kind = i % 6
    if kind == 1:
        comp = inputs.pace_params(rng, comp)
    elif kind == 2:  # tied for good
        comp[:] = [6.0, 6.0, 1.0, 0.0, 3.0]
    elif kind == 3:  # the target is behind the leader already
        state = (7, np.full(n, 60.0, np.float32), np.full(n, 5.0, np.float32))
        target = 50.0
    elif kind == 4:  # one tick from a large tick number
        state = (1 << 31, rng.uniform(0, 900, n).astype(np.float32),
                 rng.uniform(1, 9, n).astype(np.float32))
        target = float(state[1].max()) + 1.0
    elif kind == 5:  # somebody reaches the line before the target is seen
        comp[0, :2] = 1990.0, 1999.0
        target = 1980.0
    return comp, state, target


@pytest.mark.parametrize("sizes", [[1], [20, 1], [4, 5, 8, 9, 12], [16, 17, 20, 13, 3, 2, 7],
                                   list(range(1, 21)) * 3])
def test_states_of_mixed_batches(torch, orc, sizes):
    rng = np.random.default_rng(len(sizes))
    reqs = [_request(rng, n, i) for i, n in enumerate(sizes)]
    announce(f"in-play states of {len(sizes)} requests")
    B = len(reqs)
    specs = [(_bbe.Race(c, L), st, 0, 1, i, 0) for i, (c, st, _) in enumerate(reqs)]
    tick = torch.zeros(B, dtype=torch.int32, device="cuda")
    pos = torch.full((B, 20), -7.0, dtype=torch.float32, device="cuda")
    prev = torch.full((B, 20), -7.0, dtype=torch.float32, device="cuda")
    _bbe.prefix_batch(specs, np.arange(B), [t for _, _, t in reqs], 21, tick, pos, prev)
    got = tick.cpu().numpy().view(np.uint32), pos.cpu().numpy(), prev.cpu().numpy()
    for i, (comp, st, target) in enumerate(reqs):
        n = comp.shape[0]
        one = api.prefix(specs[i][0], 21, i, i, target, state=st)
        try:
            want = orc.race_prefix(comp, L, 21, i, i, np.float32(target), state=st)
        except orc.OracleError:  # somebody crossed first: the contract gives the tick only
            assert got[0][i] == 0xFFFFFFFF and one[0].item() & 0xFFFFFFFF == 0xFFFFFFFF
            continue
        for t, p, s in ((got[0][i], got[1][i, :n], got[2][i, :n]),
                        (np.uint32(one[0].item() & 0xFFFFFFFF), one[1].cpu().numpy(),
                         one[2].cpu().numpy())):
            assert t == want[0]
            np.testing.assert_array_equal(p, want[1])
            np.testing.assert_array_equal(s, want[2])
        assert not got[1][i, n:].any() and not got[2][i, n:].any()


@pytest.mark.parametrize("n", [1, 4, 8, 9, 16, 17, 20])
def test_traces_across_draw_refills(torch, orc, n):
    rng = np.random.default_rng(40 + n)
    for i, rows in enumerate((1, 2, 22, 65, 500, 500)):
        comp, state, _ = _request(rng, n, i if i < 5 else 1)
        announce(f"trace n={n} rows={rows}")
        got = api.trace(_bbe.Race(comp, L), 9, n, i, rows, state=state)
        want = orc.race_trace(comp, L, 9, n, i, rows, state=state)
        np.testing.assert_array_equal(got.cpu().numpy(), want)
