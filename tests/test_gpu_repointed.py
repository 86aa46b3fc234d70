"""Plans whose requests share waves, pointed to states of their own and back:
the items in use are those that the states call for, decided where the launch
runs (so that a captured re-pointing brings its own), and the results are those
of a plan made from these states and, in a sample, of the oracle."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from paper_2108_02419_amd import inputs
from paper_2108_02419_amd._bbe import BatchPlan, Race

pytestmark = pytest.mark.gpu
L = inputs.TRACK_LEN
SEED = 23


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def _states(orc, comp, k):
    return [orc.race_prefix(comp, L, 5, 0x80000000, s, 300.0 + 1000.0 * s / k) for s in range(k)]


def _arrays(states):
    return (np.array([s[0] for s in states], np.uint32), np.array([s[1] for s in states]),
            np.array([s[2] for s in states]))


class _Case:
    """`count` requests of `sims` simulations each (and one of 64 * big + 1 at
    either end), all from the start when the plan is made."""

    def __init__(self, torch, orc, n, count, sims, big=0, paced=False):
        rng = np.random.default_rng([n, count])
        self.comp = inputs.competitor_params(rng, n)
        if paced:
            self.comp = inputs.pace_params(rng, self.comp)
        self.n, self.orc, self.torch = n, orc, torch
        self.race = Race(self.comp, L)
        self.sims = [sims] * count
        self.sims[0] += 64 * big
        self.sims[-1] += 64 * big
        self.wins = torch.zeros((count, 20), dtype=torch.int64, device="cuda")
        self.steps = torch.zeros(1, dtype=torch.int64, device="cuda")
        self.plan = self._plan([None] * count, self.wins, self.steps)
        self.shared = self.plan.info()["n_items"]
        self.alone = sum(-(-s // 64) for s in self.sims)

    def _plan(self, states, wins, steps):
        specs = [(self.race, st, 0, m, 900 + i, 0)
                 for i, (st, m) in enumerate(zip(states, self.sims))]
        return BatchPlan(specs, SEED, wins, None, steps, autotune=False)

    def expect(self, states, what):
        """The plan's launch gives the results of these states."""
        announce(f"re-pointed n={self.n} requests={len(self.sims)}: {what}")
        for _ in range(2):
            self.plan.launch()
        w, s = self.torch.zeros_like(self.wins), self.torch.zeros_like(self.steps)
        fresh = self._plan(states, w, s)
        fresh.launch()
        self.torch.cuda.synchronize()
        assert self.torch.equal(self.wins, w) and self.torch.equal(self.steps, s)
        for i in {0, len(states) // 3, len(states) - 1}:
            _, ow, _ = self.orc.race_sim(self.comp, L, self.sims[i], SEED, request=900 + i,
                                         state=states[i], want_orders=False)
            np.testing.assert_array_equal(
                self.wins[i, :self.n].cpu().numpy().astype(np.uint64), ow)


@pytest.mark.parametrize("n,count,sims,big,paced", [(5, 64, 1, 0, False), (9, 130, 3, 2, True),
                                                    (20, 10, 1, 0, False), (20, 300, 7, 1, False)])
def test_small_plans_run_apart(torch, orc, n, count, sims, big, paced):
    c = _Case(torch, orc, n, count, sims, big, paced)
    assert c.shared < c.alone
    pool = _states(orc, c.comp, 8)
    for k in (8, 1, 2):
        states = [pool[i * k // count] for i in range(count)]
        c.plan.set_states(*_arrays(states))
        # one state: shared; more would run one after the other in a wave
        assert c.plan.info()["n_items"] == (c.shared if k == 1 else c.alone)
        c.expect(states, f"{k} states")
    states = [pool[i % 2] for i in range(count)]
    c.plan.set_states(*_arrays(states))
    assert c.plan.info()["n_items"] == c.alone
    c.expect(states, "two states in turn")


def test_large_plan_shares_as_long_as_that_is_less_work(torch, orc):
    c = _Case(torch, orc, 3, 20_000, 1)
    pool = _states(orc, c.comp, 12)
    for k in (1, 2, 12):
        states = [pool[i * k // 20_000] for i in range(20_000)]
        c.plan.set_states(*_arrays(states))
        assert c.plan.info()["n_items"] == (c.alone if k == 12 else c.shared)
        c.expect(states, f"{k} states")


def test_captured_repointing(torch, orc):
    c = _Case(torch, orc, 7, 40, 2)
    pool = _states(orc, c.comp, 40)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.plan.set_states(*_arrays(pool))
    c.expect([None] * 40, "captured, not replayed")
    for _ in range(2):
        graph.replay()
        c.expect(pool, "replayed")
    together = [pool[3]] * 40
    c.plan.set_states(*_arrays(together))
    c.expect(together, "one state again")


def test_requests_are_grouped_by_value(torch, orc):
    """Handles of equal races share waves; races that differ in one value of one
    competitor, or in the time term, do not."""
    rng = np.random.default_rng(4)
    base = inputs.pace_params(rng, inputs.competitor_params(rng, 6))
    comps = [base, base.copy()]
    for col in range(7):
        comps.append(base.copy())
        comps[-1][5, col] *= np.float32(0.99) if col != 6 else np.float32(0.5)
    comps[-1][5, 6] = np.floor(comps[-1][5, 6])
    specs = [(Race(c, L), None, 0, 3, 40 + i, 0) for i, c in enumerate(comps)]
    wins = torch.zeros((len(specs), 20), dtype=torch.int64, device="cuda")
    plan = BatchPlan(specs, SEED, wins, None, None, autotune=False)
    announce("nine races, two of them equal")
    assert plan.info()["n_items"] == len(specs) - 1
    plan.launch()
    torch.cuda.synchronize()
    for i, c in enumerate(comps):
        _, ow, _ = orc.race_sim(c, L, 3, SEED, request=40 + i, want_orders=False)
        np.testing.assert_array_equal(wins[i, :6].cpu().numpy().astype(np.uint64), ow)
