"""Requests of one race from one state share waves in a batch: counts stay
those of the oracle, for remainders below and above a wave, plain and paced
races, several races and states in one batch, and after the states of requests
that share a wave were set apart and together again.  Whole numbers, so exact.
"""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from paper_2108_02419_amd import inputs
from paper_2108_02419_amd._bbe import BatchPlan, Race

pytestmark = pytest.mark.gpu
L = inputs.TRACK_LEN
SEED = 17


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def _state(orc, comp, target):
    return orc.race_prefix(comp, L, 5, 0x80000000, 0, target)


@pytest.mark.parametrize("n,paced", [(1, False), (2, False), (7, True), (13, False), (19, True),
                                     (20, False)])
def test_requests_that_share_waves(torch, orc, n, paced):
    rng = np.random.default_rng(1000 * n + paced)
    comps = [inputs.competitor_params(rng, n), inputs.competitor_params(rng, max(1, n - 1))]
    if paced:
        comps[0] = inputs.pace_params(rng, comps[0])
    races = [Race(c, L) for c in comps]
    starts = [None if n % 2 else _state(orc, comps[0], 700.0), _state(orc, comps[1], 300.0)]
    sizes = [1, 63, 64, 65, 2, 130, 1, 1, 200, 17, 300, 5]
    which, specs = [], []
    for i in range(60):
        w = int(i % 7 == 3)
        stop = 1 if i % 11 == 5 else 0
        which.append((w, stop))
        specs.append((races[w], starts[w], 3 * i, sizes[i % len(sizes)], 500 + i, stop))

    def check(plan, wins, steps, states, what):
        announce(f"shared waves n={n} paced={paced}: {what}")
        for _ in range(2):
            plan.launch()
        torch.cuda.synchronize()
        W, total = wins.cpu().numpy(), 0
        for i, (_, _, begin, n_sims, request, stop) in enumerate(specs):
            comp = comps[which[i][0]]
            _, w, s = orc.race_sim(comp, L, n_sims, SEED, request=request, state=states[i],
                                   sim_begin=begin, stop_after=stop or comp.shape[0],
                                   want_orders=False)
            np.testing.assert_array_equal(W[i, :w.size].astype(np.uint64), w)
            assert (W[i, w.size:] == 0).all()
            total += s
        assert int(steps.item()) == total

    wins = torch.zeros((len(specs), 20), dtype=torch.int64, device="cuda")
    steps = torch.zeros(1, dtype=torch.int64, device="cuda")
    plan = BatchPlan(specs, SEED, wins, None, steps, autotune=False)
    check(plan, wins, steps, [starts[w] for w, _ in which], "as created")
    assert plan.info()["n_items"] < sum(-(-s[3] // 64) for s in specs)

    # three states among the requests of a wave, then one for each race
    apart = [[_state(orc, c, t) for t in (100.0, 900.0, 1500.0)] for c in comps]
    for what, states in (("apart", [apart[w][i % 3] for i, (w, _) in enumerate(which)]),
                         ("together", [apart[w][1] for w, _ in which])):
        tick = np.array([s[0] for s in states], np.uint32)
        pos, prev = np.zeros((60, n), np.float32), np.zeros((60, n), np.float32)
        for i, s in enumerate(states):
            pos[i, :len(s[1])], prev[i, :len(s[2])] = s[1], s[2]
        plan.set_states(tick, pos, prev)
        check(plan, wins, steps, states, what)


@pytest.mark.parametrize("split", [1, 20, 39])
def test_two_states_in_a_shared_wave(torch, orc, split):
    """Many small requests, the first `split` from one state and the others
    from another: shared waves run once for each."""
    rng = np.random.default_rng(split)
    comp = inputs.competitor_params(rng, 9)
    race = Race(comp, L)
    specs = [(race, None, 0, 1 + i % 9, 70 + i, 0) for i in range(40)]
    wins = torch.zeros((40, 20), dtype=torch.int64, device="cuda")
    steps = torch.zeros(1, dtype=torch.int64, device="cuda")
    plan = BatchPlan(specs, SEED, wins, None, steps, autotune=False)
    a, b = _state(orc, comp, 500.0), _state(orc, comp, 1100.0)
    states = [a if i < split else b for i in range(40)]
    plan.set_states(np.array([s[0] for s in states], np.uint32),
                    np.array([s[1] for s in states]), np.array([s[2] for s in states]))
    announce(f"shared waves, {split} of 40 requests in another state")
    for _ in range(2):
        plan.launch()
    torch.cuda.synchronize()
    total = 0
    for i, (_, _, _, n_sims, request, _) in enumerate(specs):
        _, w, s = orc.race_sim(comp, L, n_sims, SEED, request=request, state=states[i],
                               want_orders=False)
        np.testing.assert_array_equal(wins[i, :9].cpu().numpy().astype(np.uint64), w)
        total += s
    assert int(steps.item()) == total
