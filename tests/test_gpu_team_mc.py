"""Dry-runs with a team of lanes each and with a lane each give the same
results: around the number of simulations where one takes over from the other,
the orders, win counts and step counts of a run just above it (a lane each)
equal those of its parts (a team each), and those of the oracle in a sample."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu
from paper_2108_02419_amd import api
from paper_2108_02419_amd._bbe import Race
from paper_2108_02419_amd import inputs
from test_gpu_plain_ticks import _field

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return require_gpu()


def _line(n):
    """The most simulations of n >= 2 competitors that get a team each."""
    return n * (8192 if n <= 8 else 3200 if n <= 16 else 1500)


@pytest.mark.parametrize("n", range(2, 21))
def test_teams_and_lanes_agree(torch, orc, n):
    rng = np.random.default_rng(n)
    for i, kind in enumerate(["plain", "near_ties", "short_track", "large_previous_steps",
                              "at_the_line", "wide_steps"]):
        comp, L, state = _field(kind, n, rng)
        if (i + n) % 3 == 0:
            comp = inputs.pace_params(rng, comp, gamma_hi=0.0005)
        stop = (n, 1, max(1, n // 2))[(i + n) % 3]
        race = Race(comp, L)
        total, half = _line(n) + 1, _line(n) // 2 + 1
        announce(f"{kind} n={n} stop={stop} sims={total}")
        run = lambda sims, begin: api.mc(race, sims, 31, request=n, state=state, sim_begin=begin,
                                         stop_after=stop, want_orders=True)
        whole, parts = run(total, 5), [run(half, 5), run(total - half, 5 + half)]
        torch.cuda.synchronize()
        assert torch.equal(whole["orders"], torch.cat([p["orders"] for p in parts]))
        assert torch.equal(whole["wins"], parts[0]["wins"] + parts[1]["wins"])
        assert whole["steps"].item() == sum(p["steps"].item() for p in parts)
        oo, _, _ = orc.race_sim(comp, L, 130, 31, request=n, state=state, sim_begin=5,
                                stop_after=stop, threads=8)
        np.testing.assert_array_equal(whole["orders"][:130].cpu().numpy(), oo)


@pytest.mark.parametrize("n,sims", [(1, 1), (2, 7), (8, 9), (9, 3), (16, 5), (17, 1), (20, 3)])
def test_few_simulations_match_oracle(torch, orc, n, sims):
    rng = np.random.default_rng([n, sims])
    for stop in (1, n):
        comp, L, _ = _field("plain", n, rng)
        announce(f"few n={n} sims={sims} stop={stop}")
        out = api.mc(Race(comp, L), sims, 3, request=1, sim_begin=2**32 - sims, stop_after=stop,
                     want_orders=True)
        torch.cuda.synchronize()
        oo, ow, os_ = orc.race_sim(comp, L, sims, 3, request=1, sim_begin=2**32 - sims,
                                   stop_after=stop)
        np.testing.assert_array_equal(out["orders"].cpu().numpy(), oo)
        np.testing.assert_array_equal(out["wins"].cpu().numpy().astype(np.uint64), ow)
        assert int(out["steps"].item()) == os_
